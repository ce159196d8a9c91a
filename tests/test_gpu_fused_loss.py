"""usl_train_step's loss inside the forward kernel, where it can go wrong: labels listed twice, instances without targets,
padded fan-ins, every layout of the activations, rows in two halves, targets of one label in every instance.  The
gradient has to equal that of the separate calls bit for bit, the loss the oracle's."""
import numpy as np
import pytest

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def general_path(monkeypatch):
    """Small layers among these have a step of their own otherwise (test_gpu_step_small.py), without a loss in the forward kernel and its marks."""
    monkeypatch.setenv("USL_TUNE_SMALL", "off")


@pytest.mark.parametrize("loss_kind", [0, 1])
@pytest.mark.parametrize("m,d,k,b,storage", [
    (1000, 64, 8, 5, "f32"), (2051, 300, 33, 9, "bf16"), (2050, 10300, 5, 7, "f32"), (2050, 24000, 48, 6, "f32"),
    (2050, 41000, 64, 5, "f32"), (2050, 65536, 16, 3, "bf16"), (70000, 500, 3, 33, "f32"),
])
def test_fused_loss(orc, m, d, k, b, storage, loss_kind):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    print("fused loss", m, d, k, b, storage, loss_kind, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=820)
    idx, W, x = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg)
    rng = np.random.default_rng(5)
    lists = [rng.integers(0, m, size=n % 70 if i else 200).tolist() + [m - 1, 0, m - 1] for i, n in enumerate(rng.integers(0, 200, size=b))]
    lists[1] = []
    off = np.cumsum([0] + [len(q) for q in lists]).astype(np.int64)
    lab = np.concatenate([np.asarray(q, dtype=np.int32) for q in lists])
    scale = 1.0 / b
    d_x, d_idx, d_W, d_off, d_lab = gu.dev(x), gu.dev(idx), gu.dev(W), gu.dev(off), gu.dev(lab)
    L = usl.Layer(m, d, k, b, storage)
    ref, ref_loss = gu.empty((b, m)), gu.empty((1,))
    L.forward(d_x, d_idx, d_W, ref, b)
    (L.bce_loss_grad if loss_kind == 0 else L.sqh_loss_grad)(ref, d_off, d_lab, scale, ref, ref_loss, b)
    for with_gx in (True, False):
        W2, m1, m2 = gu.dev(W), gu.empty((m, k)).fill_(0.0), gu.empty((m, k)).fill_(0.0)
        g, gW, loss = gu.empty((b, m)), gu.empty((m, k)), gu.empty((1,))
        gx = gu.empty((b, d)) if with_gx else None
        L.train_step(d_x, d_idx, W2, m1, m2, d_off, d_lab, loss_kind, scale, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
        np.testing.assert_array_equal(gu.host(g), gu.host(ref))
        assert_close(gu.host(loss), gu.host(ref_loss), 1e-5, "loss")
        assert_close(gu.host(gW), orc.backward_weight(gu.host(g), x, idx), 1e-5, "grad_W")
    L.close()


@pytest.mark.parametrize("size", [1.0, 1e24])
@pytest.mark.parametrize("loss_kind", [0, 1])
@pytest.mark.parametrize("m,d,k,b,storage", [(5000, 300, 16, 70, "f32"), (5000, 300, 12, 37, "bf16"), (5000, 12000, 32, 34, "f32"), (2050, 24000, 32, 65, "f32")])
def test_targets_that_are_learned(orc, m, d, k, b, storage, loss_kind, size):
    """Every target far on its side of the margin, every other score far on the other: the squared hinge is exactly 0,
    also where the square of a score exceeds float32 (a target's loss must not be taken as if it were none, and then
    taken back), and the binary cross-entropy is what the separate calls give.  The batch ends off a word of 32
    instances.  Twice, the second time with other targets: what marks them does not outlive the call."""
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    print("learned targets", m, d, k, b, storage, loss_kind, size, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=830)
    idx = wl.gen_idx(cfg)
    x = wl.store(1.0 + np.abs(wl.as_f32(wl.gen_x(cfg))), storage)
    scale = 1.0 / b
    L = usl.Layer(m, d, k, b, storage)
    d_x, d_idx = gu.dev(x), gu.dev(idx)
    rng = np.random.default_rng(7)
    for turn in range(2):
        targets = rng.choice(m, size=19, replace=False).astype(np.int32)
        W = -np.abs(rng.normal(1.0, 0.2, size=(m, k))).astype(np.float32) * np.float32(3.0 if loss_kind == 0 else 1.0)
        W[targets] = np.abs(W[targets]) * np.float32(size)
        W = wl.store(W, storage)
        off, lab = np.arange(b + 1, dtype=np.int64) * 19, np.tile(targets, b)
        d_W, d_off, d_lab = gu.dev(W), gu.dev(off), gu.dev(lab)
        ref, ref_loss = gu.empty((b, m)), gu.empty((1,))
        L.forward(d_x, d_idx, d_W, ref, b)
        (L.bce_loss_grad if loss_kind == 0 else L.sqh_loss_grad)(ref, d_off, d_lab, scale, ref, ref_loss, b)
        m1, m2 = gu.empty((m, k)).fill_(0.0), gu.empty((m, k)).fill_(0.0)
        g, gW, loss = gu.empty((b, m)), gu.empty((m, k)), gu.empty((1,)).fill_(float("nan"))
        L.train_step(d_x, d_idx, d_W, m1, m2, d_off, d_lab, loss_kind, scale, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, None, loss, b)
        np.testing.assert_array_equal(gu.host(g), gu.host(ref))
        # both are float32 sums of at most 16 losses, added up in float64
        assert abs(gu.host(loss)[0] - gu.host(ref_loss)[0]) <= 1e-6 * abs(gu.host(ref_loss)[0])
        if loss_kind == 1:
            assert gu.host(loss)[0] == 0.0
    L.close()


def test_marks_of_a_step_without_gradient_do_not_stay(orc):
    """At scale 0 a target's gradient has the same bits as without the target; what marked it is cleared all the same."""
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    m, d, k, b = 3000, 300, 16, 40
    cfg = wl.custom(m, d, k, b, positives=3, index=835)
    d_idx, d_W, d_x = gu.dev(wl.gen_idx(cfg)), gu.dev(wl.gen_W(cfg)), gu.dev(wl.gen_x(cfg))
    rng = np.random.default_rng(9)
    L = usl.Layer(m, d, k, b)
    m1, m2, g, gW, loss, ref, ref_loss = (gu.empty(s).fill_(0.0) for s in [(m, k), (m, k), (b, m), (m, k), (1,), (b, m), (1,)])
    for scale in (0.0, 1.0 / b):
        off, lab = gu.dev(np.arange(b + 1, dtype=np.int64) * 7), gu.dev(rng.integers(0, m, size=7 * b).astype(np.int32))
        for loss_kind in (0, 1):
            L.forward(d_x, d_idx, d_W, ref, b)
            (L.bce_loss_grad if loss_kind == 0 else L.sqh_loss_grad)(ref, off, lab, scale, ref, ref_loss, b)
            L.train_step(d_x, d_idx, d_W, m1, m2, off, lab, loss_kind, scale, 1, 0.0, 0.9, 0.999, 1e-8, g, gW, None, loss, b)
            np.testing.assert_array_equal(gu.host(g), gu.host(ref))
            assert_close(gu.host(loss), gu.host(ref_loss), 1e-6, "loss")
    L.close()


def test_a_context_for_far_larger_batches(orc):
    """The bits that mark targets are held to 1 GiB; beyond, the loss is a pass of its own and the step gives the same."""
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    m, d, k, b = 140000, 64, 8, 5
    cfg = wl.custom(m, d, k, b, positives=3, index=836)
    idx, W, x = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg)
    off, lab = wl.gen_targets(cfg)
    d_idx, d_W, d_x, d_off, d_lab = gu.dev(idx), gu.dev(W), gu.dev(x), gu.dev(off), gu.dev(lab)
    m1, m2, g, gW, gx, loss = (gu.empty(s).fill_(0.0) for s in [(m, k), (m, k), (b, m), (m, k), (b, d), (1,)])
    L = usl.Layer(m, d, k, 65535)
    L.train_step(d_x, d_idx, d_W, m1, m2, d_off, d_lab, 0, 0.2, 1, 0.0, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
    ref_loss, ref_g = orc.bce_loss_grad(orc.forward(x, idx, W), off, lab, 0.2)
    assert_close(gu.host(g), ref_g, 1e-5, "g")
    assert abs(gu.host(loss)[0] - ref_loss) <= 1e-5 * abs(ref_loss)
    assert_close(gu.host(gW), orc.backward_weight(ref_g, x, idx), 1e-5, "grad_W")
    assert_close(gu.host(gx), orc.backward_input(ref_g, idx, W, d), 1e-4, "grad_x")
    L.close()


@pytest.mark.parametrize("m,d,k,b,storage", [(3001, 300, 32, 21, "f32"), (2049, 9000, 8, 18, "bf16"), (2050, 24000, 48, 19, "f32"), (1500, 50000, 33, 17, "f32")])
@pytest.mark.parametrize("factor", [0.0, 0.01, 1.0, 12.0, 60.0])
def test_loss_of_small_and_large_scores(m, d, k, b, storage, factor):
    """The loss inside forward against float64 of the same scores.  A score's terms carry two roundings of the hardware's exponential and logarithm (an
    ulp each) and those of up to four scores' sums, at most 8 * 2^-24 of the terms' magnitude together; everything else is float64: 1e-6."""
    import gpu_util as gu
    import torch
    from paper_2306_03725_amd import usl
    print("loss of scores", m, d, k, b, storage, factor, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=821)
    idx, x = wl.gen_idx(cfg), wl.gen_x(cfg)
    W = wl.store(wl.as_f32(wl.gen_W(cfg)) * np.float32(factor), storage)
    off = np.arange(b + 1, dtype=np.int64) * 3
    lab = np.stack([np.random.default_rng(i).choice(m, 3, replace=False) for i in range(b)]).astype(np.int32).reshape(-1)
    d_x, d_idx, d_W, d_off, d_lab = gu.dev(x), gu.dev(idx), gu.dev(W), gu.dev(off), gu.dev(lab)
    L = usl.Layer(m, d, k, b, storage)
    z = gu.empty((b, m))
    L.forward(d_x, d_idx, d_W, z, b)
    z64, y = gu.host(z).astype(np.float64), np.zeros((b, m))
    y[np.repeat(np.arange(b), 3), lab] = 1.0
    terms = np.maximum(z64, 0.0) - z64 * y + np.log1p(np.exp(-np.abs(z64)))
    g, gW, gx, loss, m1, m2 = gu.empty((b, m)), gu.empty((m, k)), gu.empty((b, d)), gu.empty((1,)), gu.empty((m, k)).zero_(), gu.empty((m, k)).zero_()
    L.train_step(d_x, d_idx, d_W, m1, m2, d_off, d_lab, 0, 1.0 / b, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
    torch.cuda.synchronize()
    magnitude = (np.maximum(z64, 0.0) + np.abs(z64) * y + np.log1p(np.exp(-np.abs(z64)))).sum() / b
    assert abs(float(gu.host(loss)[0]) - terms.sum() / b) <= 1e-6 * magnitude
    L.close()


# (The bound of the test above leaves out the rounding of 1 + e, which is 2^-24 of the term's own size or absolutely, whichever is more.  It holds there because those scores lie
# on both sides of 0: a score's magnitude is 0.3 or more on average, and all roundings together stay below 16 * 2^-24 of it.)
@pytest.mark.parametrize("m,d,k,b,storage", [(3001, 300, 32, 21, "f32"), (2049, 9000, 8, 18, "bf16"), (2050, 24000, 48, 19, "f32"), (1500, 50000, 33, 17, "f32")])
@pytest.mark.parametrize("mean", [-4.5, -10.0, -14.0, -17.0, -40.0])
def test_loss_of_scores_that_are_all_negative(m, d, k, b, storage, mean):
    """A trained layer without a target among its scores: every term is log(1 + e) of a small e.  1 + e is rounded to 2^-24 (all of an e below that is lost),
    the logarithm of what is left to an ulp of itself: at most 2^-24 + 8 * 2^-24 of the term for a score, whatever the term is.  The sum over instances is divided by b."""
    import gpu_util as gu
    import torch
    from paper_2306_03725_amd import usl
    print("loss of negative scores", m, d, k, b, storage, mean, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=822)
    idx, x = wl.gen_idx(cfg), wl.gen_x(cfg)
    W = wl.store((mean / (0.4 * k) * (1.0 + 0.1 * np.random.default_rng(5).standard_normal((m, k)))).astype(np.float32), storage)
    d_x, d_idx, d_W, d_off, d_lab = gu.dev(x), gu.dev(idx), gu.dev(W), gu.dev(np.zeros(b + 1, dtype=np.int64)), gu.dev(np.zeros(1, dtype=np.int32))
    L = usl.Layer(m, d, k, b, storage)
    z = gu.empty((b, m))
    L.forward(d_x, d_idx, d_W, z, b)
    z64 = gu.host(z).astype(np.float64)
    assert (z64 <= 0.0).all()
    terms = np.log1p(np.exp(z64)).sum() / b
    g, gW, gx, loss, m1, m2 = gu.empty((b, m)), gu.empty((m, k)), gu.empty((b, d)), gu.empty((1,)), gu.empty((m, k)).zero_(), gu.empty((m, k)).zero_()
    L.train_step(d_x, d_idx, d_W, m1, m2, d_off, d_lab, 0, 1.0 / b, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
    torch.cuda.synchronize()
    assert abs(float(gu.host(loss)[0]) - terms) <= 2.0 ** -24 * m + 8 * 2.0 ** -24 * terms
    L.close()
