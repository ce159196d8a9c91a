"""Prediction (Section 2): top-k labels of the score rows and the precision-at-k hit counts, HIP path
(through the C ABI) against the CPU oracle.  Integer and index work: bit-exact."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def usl():
    from paper_2306_03725_amd import usl as u
    assert torch.cuda.is_available()
    return u


@pytest.fixture(scope="module")
def gu():
    import gpu_util
    return gpu_util


def run_topk(usl, gu, orc, scores, kk):
    b, m = scores.shape
    L = usl.Layer(m, 1, 1, b)
    lab = gu.empty((b, kk), torch.int32).fill_(-7)
    val = gu.empty((b, kk)).fill_(float("nan"))
    L.topk(gu.dev(scores), b, kk, lab, val)
    ref_lab, ref_val = orc.topk(scores, kk)
    np.testing.assert_array_equal(gu.host(lab), ref_lab)
    np.testing.assert_array_equal(gu.host(val).view(np.uint32), ref_val.view(np.uint32))
    return lab, ref_lab


# (m, b, kk): one segment; a ragged second segment; exactly one / one more than a segment; kk == m;
# several segments with the largest kk
TOPK_CASES = [(1024, 16, 5), (30938, 7, 3), (16384, 3, 1), (16385, 3, 32), (5, 4, 5), (1, 2, 1),
              (100000, 5, 32), (40, 3, 32)]


@pytest.mark.parametrize("m,b,kk", TOPK_CASES)
def test_topk_random_scores(usl, gu, orc, m, b, kk):
    print("topk", m, b, kk, flush=True)
    r = np.random.default_rng([m, b, kk])
    scores = (r.standard_normal((b, m)) * 3).astype(np.float32)
    run_topk(usl, gu, orc, scores, kk)


@pytest.mark.parametrize("m,b,kk", [(3000, 6, 17), (50000, 4, 32), (16390, 2, 8)])
def test_topk_ties_zeros_infinities(usl, gu, orc, m, b, kk):
    """Few distinct values: the order inside a tie is by label; -0 and +0 tie; infinities are scores."""
    r = np.random.default_rng([m, kk, 3])
    scores = r.integers(-2, 3, size=(b, m)).astype(np.float32)
    zeros = scores == 0
    scores[zeros] *= r.choice([-1.0, 1.0], size=int(zeros.sum())).astype(np.float32)
    scores[0, r.integers(0, m, 3)] = np.inf
    scores[1, :] = -np.inf                       # a whole row of equal scores: labels 0..kk-1
    scores[2 % b, m - 1] = 100.0                 # the very last label wins
    if b > 3:
        scores[3] = -0.0                         # all zeros of one sign ...
        scores[3, 1::2] = 0.0                    # ... and the other: still one tie
    run_topk(usl, gu, orc, scores, kk)


def test_topk_all_in_one_lane(usl, gu, orc):
    """The kk best scores all sit in labels that one lane of the workgroup reads (stride 256)."""
    m, b, kk = 40000, 2, 32
    scores = np.random.default_rng(4).standard_normal((b, m)).astype(np.float32)
    scores[0, 5::256][:60] += 50.0
    scores[1, 16384 + 255::256][:40] += 50.0
    run_topk(usl, gu, orc, scores, kk)


@pytest.mark.parametrize("name", ["tiny", "medium"])
def test_precision_hits(usl, gu, orc, name):
    cfg = wl.CONFIGS[name]
    m, b, kk = cfg.m, cfg.b, 5
    off, lab = wl.gen_targets(cfg)
    r = wl.rng(cfg, 31)
    scores = r.standard_normal((b, m)).astype(np.float32)
    for i in range(b):                            # lift some of every instance's targets into the top
        t = lab[off[i]:off[i + 1]]
        scores[i, t[: 1 + i % 3]] += 6.0
    top, ref_top = run_topk(usl, gu, orc, scores, kk)
    L = usl.Layer(m, cfg.d, cfg.k, b)
    hits = gu.empty((kk,), torch.int64).fill_(-1)
    L.precision_hits(top, gu.dev(off), gu.dev(lab), b, kk, hits)
    ref = orc.precision_hits(ref_top, off, lab)
    np.testing.assert_array_equal(gu.host(hits), ref)
    assert ref.sum() > 0
    L.precision_hits(top, gu.dev(off), gu.dev(lab), b, kk, hits)      # overwritten, not accumulated
    np.testing.assert_array_equal(gu.host(hits), ref)


def test_topk_argument_errors(usl, gu):
    L = usl.Layer(100, 10, 2, 4)
    out = gu.empty((4, 100)).zero_()
    lab, val = gu.empty((4, 40), torch.int32), gu.empty((4, 40))
    for kk, status in ((0, 1), (33, 2), (101, 2)):
        with pytest.raises(usl.UslError) as e:
            L.topk(out, 4, kk, lab, val)
        assert e.value.status == status
    with pytest.raises(usl.UslError):
        L.topk(out, 5, 3, lab, val)              # batch beyond max_b


@pytest.mark.parametrize("m,d,k,b,kk,storage", [(1024, 64, 8, 16, 5, "f32"), (30938, 1024, 32, 70, 3, "f32"),
                                                (3001, 1000, 32, 37, 32, "bf16"), (270001, 2048, 32, 33, 5, "f32"),
                                                (500, 203, 5, 65, 1, "f32")])
def test_predict_is_forward_then_topk(usl, gu, orc, m, d, k, b, kk, storage):
    """usl_predict (scores through library scratch) against the oracle's top-k of the scores the forward call
    writes, and those scores against the oracle's."""
    _predict_case(usl, gu, orc, m, d, k, b, kk, storage)


def test_predict_in_chunks(usl, gu, orc, monkeypatch):
    """A scratch cap of 70 rows: 150 instances go through as 70 + 70 + 10; a cap below 64 rows means 64."""
    m = 30938
    monkeypatch.setenv("USL_TUNE_PREDICT_BYTES", str(70 * m * 4))
    _predict_case(usl, gu, orc, m, 1024, 32, 150, 5, "f32")
    monkeypatch.setenv("USL_TUNE_PREDICT_BYTES", str(3 * m * 4))
    _predict_case(usl, gu, orc, m, 1024, 32, 130, 2, "f32")


def _predict_case(usl, gu, orc, m, d, k, b, kk, storage):
    from helpers import assert_close
    cfg = wl.custom(m, d, k, b, storage=storage, positives=1, index=150)
    idx, W, x = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg)
    L = usl.Layer(m, d, k, b, storage)
    d_idx, d_W, d_x = gu.dev(idx), gu.dev(W), gu.dev(x)
    lab, val = gu.empty((b, kk), torch.int32).fill_(-1), gu.empty((b, kk)).fill_(float("nan"))
    L.predict(d_x, d_idx, d_W, b, kk, lab, val)
    out = gu.empty((b, m))
    L.forward(d_x, d_idx, d_W, out, b)
    scores = gu.host(out)
    assert_close(scores, orc.forward(x, idx, W), 1e-5, "scores")
    ref_lab, ref_val = orc.topk(scores, kk)
    np.testing.assert_array_equal(gu.host(lab), ref_lab)
    np.testing.assert_array_equal(gu.host(val).view(np.uint32), ref_val.view(np.uint32))


# One instance, forward and the selection in one kernel or, for layers in between, in several: turns of a wavefront beyond those it keeps in registers (five: rows of
# which a compute unit holds one, m = 1.2 million), workgroups of 4 to 16 wavefronts, the last one ragged, fewer labels than kk to a workgroup, ties.  Two to four instances: the
# streaming forward, then the selection
@pytest.mark.parametrize("m,d,k,b,kk,storage", [
    (5, 8, 3, 1, 5, "f32"), (33, 8, 2, 4, 32, "f32"), (1000, 100, 8, 2, 7, "bf16"), (70001, 300, 33, 3, 32, "f32"), (300001, 64, 8, 4, 5, "f32"),
    (2000003, 64, 4, 1, 32, "f32"), (500000, 32768, 32, 1, 5, "f32"), (131072, 20000, 16, 2, 1, "bf16"), (200000, 40000, 5, 1, 32, "bf16"),
    (1200001, 21000, 4, 1, 9, "f32"), (225711, 118, 13, 1, 5, "f32"), (1050075, 597, 8, 1, 5, "bf16"), (60867, 300, 16, 1, 32, "f32")])
def test_predict_of_one_group(usl, gu, orc, m, d, k, b, kk, storage):
    print("predict of one group", m, d, k, b, kk, storage, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=min(3, m), index=870)
    idx, x = wl.gen_idx(cfg), wl.gen_x(cfg)
    W = wl.store(np.round(wl.as_f32(wl.gen_W(cfg)) * 4) / 4, storage)      # few values: many scores are alike
    x = wl.store(np.round(wl.as_f32(x)), storage)
    if m == 1200001:   # the best labels in a wavefront's last turn, whose scores it reads back
        x, W = np.abs(x), wl.as_f32(W)
        W[m - 5000:m - 4900] = 9.0
    L = usl.Layer(m, d, k, b, storage)
    d_x, d_idx, d_W = gu.dev(x), gu.dev(idx), gu.dev(W)
    out = gu.empty((b, m))
    L.forward(d_x, d_idx, d_W, out, b)
    if m == 1200001:
        assert (orc.topk(gu.host(out), kk)[0] >= m - 5000).all()
    ref_lab, ref_val = orc.topk(gu.host(out), kk)
    for n in (kk, max(1, kk // 2)):
        lab, val = gu.empty((b, n), torch.int32).fill_(-1), gu.empty((b, n)).fill_(float("nan"))
        L.predict(d_x, d_idx, d_W, b, n, lab, val)
        np.testing.assert_array_equal(gu.host(lab), ref_lab[:, :n])
        np.testing.assert_array_equal(gu.host(val).view(np.uint32), np.ascontiguousarray(ref_val[:, :n]).view(np.uint32))
    L.close()


@pytest.mark.parametrize("m,d,k", [(500000, 32768, 32), (4097, 64, 8), (60867, 1344, 16)])
def test_merge_by_the_workgroup_that_comes_last(usl, gu, orc, m, d, k):
    """Calls one behind the other with other inputs and other numbers of labels (beyond some the merge is a launch of its own), then the same from a
    captured graph: the count of finished workgroups is 0 again after every call."""
    print("merge", m, d, k, flush=True)
    cfg = wl.custom(m, d, k, 8, positives=1, index=871)
    x = wl.gen_x(cfg)
    L = usl.Layer(m, d, k, 8, stream=torch.cuda.current_stream().cuda_stream)
    d_idx, d_W, d_out = gu.dev(wl.gen_idx(cfg)), gu.dev(wl.gen_W(cfg)), gu.empty((1, m))
    rows, want, got = [gu.dev(x[i:i + 1]) for i in range(8)], [], []
    for row in rows:
        L.forward(row, d_idx, d_W, d_out, 1)
        want.append(orc.topk(gu.host(d_out), 32))
    for i in range(24):
        kk = (5, 32, 1, 16)[i % 4]
        lab, val = gu.empty((1, kk), torch.int32).fill_(-1), gu.empty((1, kk))
        L.predict(rows[i % 8], d_idx, d_W, 1, kk, lab, val)
        got.append((i % 8, kk, lab, val))
    for i, kk, lab, val in got:
        np.testing.assert_array_equal(gu.host(lab), want[i][0][:, :kk])
        np.testing.assert_array_equal(gu.host(val).view(np.uint32), np.ascontiguousarray(want[i][1][:, :kk]).view(np.uint32))
    stream, row, lab, val = torch.cuda.Stream(), rows[0].clone(), gu.empty((1, 5), torch.int32), gu.empty((1, 5))
    torch.cuda.synchronize()
    L.set_stream(stream.cuda_stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        L.predict(row, d_idx, d_W, 1, 5, lab, val)
    for i in (3, 5, 1):
        row.copy_(rows[i])
        graph.replay()
        np.testing.assert_array_equal(gu.host(lab), want[i][0][:, :5])
        (row + 1).sum().item()
    L.close()


# Merged by the last workgroup: 256 of 16 wavefronts for 5, 1 and 16 labels, 17 of 4 wavefronts for all.  A launch of its own: 32 labels of the former.  (In the test above
# (60867, 1344, 16) never merges that way: 476 workgroups.)
@pytest.mark.parametrize("m,d,k,storage", [(500000, 32768, 32, "f32"), (4097, 64, 8, "f32"), (4097, 64, 8, "bf16"), (300001, 60000, 32, "bf16")])
def test_scores_of_merges_by_the_workgroup_that_comes_last(usl, gu, orc, m, d, k, storage):
    """Labels and the bits of the scores, of calls one behind the other and of every replay, into arrays that hold something else."""
    print("scores of merges", m, d, k, storage, flush=True)
    cfg = wl.custom(m, d, k, 8, storage=storage, positives=1, index=871)
    x = wl.gen_x(cfg)
    L = usl.Layer(m, d, k, 8, storage, torch.cuda.current_stream().cuda_stream)
    d_idx, d_W, d_out = gu.dev(wl.gen_idx(cfg)), gu.dev(wl.gen_W(cfg)), gu.empty((1, m))
    rows, want = [gu.dev(x[i:i + 1]) for i in range(8)], []
    for row in rows:
        L.forward(row, d_idx, d_W, d_out, 1)
        want.append(orc.topk(gu.host(d_out), 32))

    def same(i, kk, lab, val):
        np.testing.assert_array_equal(gu.host(lab), want[i][0][:, :kk])
        np.testing.assert_array_equal(gu.host(val).view(np.uint32), np.ascontiguousarray(want[i][1][:, :kk]).view(np.uint32))

    got = []
    for i in range(24):
        kk = (5, 32, 1, 16)[i % 4]
        lab, val = gu.empty((1, kk), torch.int32).fill_(-1), gu.empty((1, kk)).fill_(-1.0)
        L.predict(rows[i % 8], d_idx, d_W, 1, kk, lab, val)
        got.append((i % 8, kk, lab, val))
    for call in got:
        same(*call)
    stream, row, lab, val = torch.cuda.Stream(), rows[0].clone(), gu.empty((1, 5), torch.int32), gu.empty((1, 5))
    torch.cuda.synchronize()
    L.set_stream(stream.cuda_stream)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        L.predict(row, d_idx, d_W, 1, 5, lab, val)
    for i in (3, 5, 1):
        row.copy_(rows[i])
        lab.fill_(-1), val.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        same(i, 5, lab, val)
        (row + 1).sum().item()
    L.close()


@pytest.mark.parametrize("first", ["plain", "captured"])
@pytest.mark.parametrize("m,d,k,storage", [(500000, 32768, 32, "f32"), (4097, 64, 8, "bf16")])
def test_capture_of_the_first_prediction_of_one_instance(usl, gu, orc, m, d, k, storage, first):
    """A context that has only predicted batches is captured, and a new one in the mode that lets a capture allocate; then plain calls before
    the first replay, and replays between plain calls: labels and the scores' bits are those of forward and the oracle's search."""
    print("first prediction captured", m, d, k, storage, first, flush=True)
    cfg = wl.custom(m, d, k, 8, storage=storage, positives=1, index=872)
    x = wl.gen_x(cfg)
    stream = torch.cuda.Stream()
    L, F = usl.Layer(m, d, k, 8, storage, stream.cuda_stream), usl.Layer(m, d, k, 8, storage)
    d_x, d_idx, d_W, d_out = gu.dev(x), gu.dev(wl.gen_idx(cfg)), gu.dev(wl.gen_W(cfg)), gu.empty((8, m))
    rows, want = [gu.dev(x[i:i + 1]) for i in range(4)], []
    for row in rows:
        F.forward(row, d_idx, d_W, d_out, 1)
        want.append(orc.topk(gu.host(d_out)[:1], 5))
    F.forward(d_x, d_idx, d_W, d_out, 8)
    ref8 = orc.topk(gu.host(d_out), 32)
    row, lab, val = rows[0].clone(), gu.empty((1, 5), torch.int32), gu.empty((1, 5))
    lab2, val2 = gu.empty((1, 5), torch.int32), gu.empty((1, 5))
    torch.cuda.synchronize()

    def same(i, labels, scores):
        stream.synchronize()
        np.testing.assert_array_equal(gu.host(labels), want[i][0])
        np.testing.assert_array_equal(gu.host(scores).view(np.uint32), want[i][1].view(np.uint32))

    with torch.cuda.stream(stream):
        if first == "plain":
            lab8, val8 = gu.empty((8, 32), torch.int32), gu.empty((8, 32))
            L.predict(d_x, d_idx, d_W, 8, 32, lab8, val8)
            stream.synchronize()
            np.testing.assert_array_equal(gu.host(lab8), ref8[0])
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream, capture_error_mode="global" if first == "plain" else "relaxed"):
            L.predict(row, d_idx, d_W, 1, 5, lab, val)
        for i in (2, 1):
            L.predict(rows[i], d_idx, d_W, 1, 5, lab2.fill_(-1), val2)
            same(i, lab2, val2)
        for i in (3, 0, 2):
            row.copy_(rows[i])
            lab.fill_(-1)
            graph.replay()
            same(i, lab, val)
            L.predict(rows[1], d_idx, d_W, 1, 5, lab2.fill_(-1), val2)
            same(1, lab2, val2)
    L.close()
    F.close()


@pytest.mark.parametrize("m,d,k", [(500000, 32768, 32), (4097, 64, 8), (30000, 64, 8)])
def test_predictions_that_overlap_spoil_no_later_one(usl, gu, orc, m, d, k):
    """Two graphs of one context replayed on two streams at a time: what they write is undefined, what calls after a wait write is not."""
    print("overlapping predictions", m, d, k, flush=True)
    cfg = wl.custom(m, d, k, 4, positives=1, index=873)
    x = wl.gen_x(cfg)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    L = usl.Layer(m, d, k, 1, stream=torch.cuda.current_stream().cuda_stream)
    d_idx, d_W, d_out = gu.dev(wl.gen_idx(cfg)), gu.dev(wl.gen_W(cfg)), gu.empty((1, m))
    rows, want = [gu.dev(x[i:i + 1]) for i in range(4)], []
    for row in rows:
        L.forward(row, d_idx, d_W, d_out, 1)
        want.append(orc.topk(gu.host(d_out), 5))
    lab, val = gu.empty((1, 5), torch.int32), gu.empty((1, 5))
    L.predict(rows[0], d_idx, d_W, 1, 5, lab, val)
    torch.cuda.synchronize()
    graphs, spare = [], [(gu.empty((1, 5), torch.int32), gu.empty((1, 5))) for _ in streams]
    for stream, to in zip(streams, spare):
        graphs.append(torch.cuda.CUDAGraph())
        L.set_stream(stream.cuda_stream)
        with torch.cuda.graph(graphs[-1], stream=stream):
            for _ in range(50):
                L.predict(rows[0], d_idx, d_W, 1, 5, *to)
    L.set_stream(torch.cuda.current_stream().cuda_stream)
    for turn in range(20):
        for stream, graph in zip(streams, graphs):
            with torch.cuda.stream(stream):
                graph.replay()
        torch.cuda.synchronize()
        for i in (1, 2, 3):
            lab.fill_(-1), val.fill_(-1.0)
            L.predict(rows[i], d_idx, d_W, 1, 5, lab, val)
            np.testing.assert_array_equal(gu.host(lab), want[i][0])
            np.testing.assert_array_equal(gu.host(val).view(np.uint32), want[i][1].view(np.uint32))
    L.close()
