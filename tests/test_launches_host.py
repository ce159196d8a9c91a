"""What the library does around its launches, with a HIP runtime that launches nothing (stand_in_hip.cpp), on the host: a refused launch leaves no marks that
the next step takes for targets, arrays that are not aligned are refused before anything is launched, a split of the batch asked for by hand that
there is no room for is a smaller one, and the count by which a prediction's last workgroup knows itself is there, and 0, before any launch that uses it."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# x, idx, W, m1, m2, tgt_off, tgt_lab, g, grad_W, grad_x, loss: addresses that nobody follows
HEAD = """
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
hip.stand_in_launched.restype = ctypes.c_char_p
sys.path.insert(0, %r)
from paper_2306_03725_amd import usl
P = dict(x=1 << 20, idx=2 << 20, W=3 << 20, m1=4 << 20, m2=5 << 20, off=6 << 20, lab=7 << 20, g=8 << 20, grad_W=9 << 20, grad_x=10 << 20, loss=11 << 20)
def step(L, b, refuse="", kind=0, **other):
    p = dict(P, **other)
    hip.stand_in_start(refuse.encode())
    status = 0
    try:
        L.train_step(p["x"], p["idx"], p["W"], p["m1"], p["m2"], p["off"], p["lab"], kind, 1.0, 1, 1e-3, 0.9, 0.999, 1e-8, p["g"], p["grad_W"], p["grad_x"], p["loss"], b)
    except usl.UslError as e:
        status = e.status
    return status, hip.stand_in_launched().decode().split()
def at(names, part):
    return [n for n, name in enumerate(names) if part in name]
""" % ROOT


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("hip") / "libstandin.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "stand_in_hip.cpp"), "-o", so])
    return so


def run(stand_in, text):
    r = subprocess.run([sys.executable, "-c", HEAD + text, stand_in], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("adam,grad_x", [("k_adam_staged", "P['grad_x']"), ("k_adam", "None")])
def test_marks_of_a_step_whose_last_launch_is_refused_are_cleared(stand_in, adam, grad_x):
    run(stand_in, """
L = usl.Layer(70000, 512, 16, 40)
s, names = step(L, 40, grad_x={gx})
assert s == 0 and at(names, "k_forward") and at(names, "{adam}"), names
assert at(names, "k_fill_zero"), names            # new scratch
s, names = step(L, 40, grad_x={gx})
assert s == 0 and not at(names, "k_fill_zero"), names
s, names = step(L, 40, refuse="{adam}", grad_x={gx})
assert s == usl.USL_EHIP, s
s, names = step(L, 40, grad_x={gx})
assert s == 0 and at(names, "k_fill_zero") and at(names, "k_fill_zero")[0] < at(names, "k_forward")[0], names
""".format(adam=adam, gx=grad_x))

def test_arrays_that_are_not_aligned_are_refused_before_a_launch(stand_in):
    run(stand_in, """
for shape in ((1024, 64, 8, 16, "f32"), (1000, 64, 4, 3, "bf16"), (70000, 512, 16, 40, "f32"), (3000, 70000, 8, 5, "f32")):
    for kind in (0, 1):
        L = usl.Layer(*shape)
        for grad_x in (P["grad_x"], None):
            for name in ("W", "m1", "m2", "grad_W"):
                s, names = step(L, shape[3], kind=kind, **{"grad_x": grad_x, name: P[name] + 4})
                assert s == usl.USL_EINVAL and not names, (shape, kind, name, s, names)
            s, names = step(L, shape[3], kind=kind, grad_x=grad_x)
            assert s == 0 and names, (shape, kind, s)
""")


def test_a_split_asked_for_that_there_is_no_room_for(stand_in):
    run(stand_in, """
import os
for split in ("2", "32", "1000"):
    os.environ["USL_TUNE_SPLIT"] = split
    L = usl.Layer(3000000, 16384, 64, 512)    # one part of the weight gradient takes more than the partial sums may
    hip.stand_in_start(b"")
    L.backward_weight(P["g"], P["x"], P["idx"], P["grad_W"], 512)
    names = hip.stand_in_launched().decode().split()
    assert at(names, "k_backward_weight") and not at(names, "k_sum_parts"), names
    L = usl.Layer(30000, 1000, 16, 512)
    hip.stand_in_start(b"")
    L.backward_weight(P["g"], P["x"], P["idx"], P["grad_W"], 512)
    assert at(hip.stand_in_launched().decode().split(), "k_sum_parts")
""")


# m, d, k, storage: one workgroup of 16 wavefronts to a compute unit; smaller workgroups; bfloat16
ONE = [(500000, 32768, 32, "f32"), (4097, 64, 8, "f32"), (4097, 64, 8, "bf16")]
PREDICT = """
def predict(L, b, kk, refuse="", capture=False):
    hip.stand_in_start(refuse.encode())
    hip.stand_in_capture(capture)
    status = 0
    try:
        L.predict(P["x"], P["idx"], P["W"], b, kk, P["off"], P["g"])
    except usl.UslError as e:
        status = e.status
    return status, hip.stand_in_launched().decode().split(), hip.stand_in_allocated()
L = usl.Layer(%d, %d, %d, 8, "%s")
"""


@pytest.mark.parametrize("shape", ONE)
def test_a_prediction_of_one_instance_finds_its_scratch(stand_in, shape):
    """Whatever the batch and kk of the first prediction were, no later one allocates or clears (it may be captured)."""
    run(stand_in, PREDICT % shape + """
s, names, n = predict(L, 8, 32)
assert s == 0 and n and at(names, "k_zero_hits"), names
for kk in (32, 5, 1):
    s, names, n = predict(L, 1, kk, capture=kk == 5)
    assert s == 0 and at(names, "k_forward_few") and not at(names, "k_zero_hits") and n == 0, (kk, names, n)
    assert kk == 32 or not at(names, "k_topk_merge"), (kk, names)
""")


# labels, features, fan-in, labels asked for; whether the last workgroup merges: few workgroups (47, 48 and 64 with 1 label, 112 and 113 with 5), 256 of 8 wavefronts, of 16 with a
# short stream, with many candidates, with too many, with a long stream, two workgroups to a compute unit
MERGES = [(12000, 600, 8, 1, True), (12288, 600, 8, 1, True), (12289, 600, 8, 1, False), (28672, 600, 8, 5, True), (28673, 600, 8, 5, False),
          (131000, 25000, 16, 5, False), (113590, 34460, 32, 5, False), (113590, 34460, 32, 8, False), (113590, 34460, 32, 9, True),
          (113590, 34460, 32, 16, True), (113590, 34460, 32, 17, False), (175219, 33043, 32, 1, True), (500000, 32768, 32, 16, True), (1340000, 11000, 3, 5, False)]


@pytest.mark.parametrize("m,d,k,kk,last", MERGES)
def test_who_merges_the_candidates(stand_in, m, d, k, kk, last):
    run(stand_in, PREDICT % (m, d, k, "f32") + """
s, names, n = predict(L, 1, %d)
assert s == 0 and at(names, "k_forward_few") and bool(at(names, "k_topk_merge")) != %r, names
""" % (kk, last))


@pytest.mark.parametrize("shape", ONE)
def test_a_count_whose_clearing_is_refused_is_cleared_by_the_next_call(stand_in, shape):
    run(stand_in, PREDICT % shape + """
s, names, n = predict(L, 1, 5, refuse="k_zero_hits")
assert s == usl.USL_EHIP and not at(names, "k_forward_few"), (s, names)
s, names, n = predict(L, 1, 5)
assert s == 0 and at(names, "k_zero_hits") and at(names, "k_zero_hits")[0] < at(names, "k_forward_few")[0], names
s, names, n = predict(L, 1, 5)
assert s == 0 and not at(names, "k_zero_hits") and not at(names, "k_topk_merge"), names
""")


@pytest.mark.parametrize("shape", ONE)
def test_a_clearing_that_is_only_recorded_does_not_count(stand_in, shape):
    """The first predictions of a context under a capture: they use no count, and the first plain call clears it before it does."""
    run(stand_in, PREDICT % shape + """
for kk in (5, 1):
    s, names, n = predict(L, 1, kk, capture=True)
    assert s == 0 and at(names, "k_forward_few") and not at(names, "k_zero_hits") and at(names, "k_topk_merge"), (kk, names)
s, names, n = predict(L, 1, 5)
assert s == 0 and n == 0 and not at(names, "k_topk_merge"), (names, n)
assert at(names, "k_zero_hits") and at(names, "k_zero_hits")[0] < at(names, "k_forward_few")[0], names
s, names, n = predict(L, 1, 5, capture=True)
assert s == 0 and n == 0 and not at(names, "k_zero_hits") and not at(names, "k_topk_merge"), (names, n)
""")


# labels, features, fan-in, labels asked for; whether the forward kernel looks for the best ones: workgroups of 4 wavefronts, 5 and 6 labels of 424, 8 of
# as many as a short merge holds and of one more, 32 of many with the pass's candidates too many for a short merge as well; one of 16 wavefronts to a compute unit, two, two with three turns
FROM_FORWARD = [(5000, 64, 8, 32, True), (54181, 600, 16, 5, True), (54181, 600, 16, 6, False), (65536, 600, 8, 8, True), (65537, 600, 8, 8, False), (60867, 1344, 16, 32, False), (262000, 25000, 8, 32, True), (200460, 188, 8, 32, False),
                (113590, 34460, 32, 32, True), (109071, 7213, 32, 1, False), (1270000, 11000, 32, 32, True)]


@pytest.mark.parametrize("m,d,k,kk,forward", FROM_FORWARD)
def test_where_the_best_labels_come_from(stand_in, m, d, k, kk, forward):
    run(stand_in, PREDICT % (m, d, k, "f32") + """
s, names, n = predict(L, 1, %d)
assert s == 0 and at(names, "k_forward_few") and bool(at(names, "k_topk_segments")) != %r, names
""" % (kk, forward))
