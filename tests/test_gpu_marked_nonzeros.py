"""usl_train_step with the squared hinge where few nonzeros are expected: forward marks them, one bit per score, and the lists of the backward
products come from the marks.  Where that can go wrong: last words and wavefronts that are not full, blocks of labels that begin at odd
multiples of 32, one, two and four instances a read, rows in two halves, batches in parts, an instance without a nonzero, one with more than a
list holds (the dense kernels then do the work).  Gradients against the oracle on the same g."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("crowded", [False, True])
@pytest.mark.parametrize("m,d,k,b,storage,env", [
    (65569, 300, 8, 5, "f32", {}), (65536, 300, 8, 34, "bf16", {}), (70001, 12000, 8, 6, "f32", {"USL_TUNE_LABELS": "96"}),
    (70031, 500, 16, 9, "f32", {"USL_TUNE_LABELS": "800"}), (65600, 32768, 8, 3, "f32", {"USL_TUNE_SPLIT": "2"}), (66001, 41000, 8, 3, "f32", {}),
    (66049, 24000, 8, 7, "bf16", {"USL_TUNE_TAIL": "2"}), (70001, 60000, 3, 5, "bf16", {})])
def test_gradients_from_marks(orc, m, d, k, b, storage, env, crowded, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SPARSE", "always")
    for name, v in env.items():
        monkeypatch.setenv(name, v)
    print("marked nonzeros", m, d, k, b, storage, env, crowded, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=995)
    idx = wl.gen_idx(cfg)
    x = np.float32(1.0) + np.abs(wl.as_f32(wl.gen_x(cfg)))
    x[1] *= 1e3                                  # every negative weight leads past the margin
    rng = np.random.default_rng(3)
    W = -np.abs(rng.normal(1.0, 0.2, size=(m, k))).astype(np.float32)
    W[rng.choice(m, size=m // 200, replace=False)] *= np.float32(-0.05)
    W[[0, 31, 32, 63, 64, m - 1]] = np.float32(0.01)
    if crowded:
        W[: m // 20] = np.float32(-0.02)         # more than m / 32 nonzeros, but for instance 1
    x, W = wl.store(x, storage), wl.store(W, storage)
    off, lab = np.arange(b + 1, dtype=np.int64) * 2, np.tile(np.array([5, m - 1], np.int32), b)
    scale = float(np.float32(1.0 / b))
    L = usl.Layer(m, d, k, b, storage)
    d_x, d_idx, d_off, d_lab = gu.dev(x), gu.dev(idx), gu.dev(off), gu.dev(lab)
    m1, m2, g, gW, gx, loss = (gu.empty(s).fill_(float("nan")) for s in [(m, k), (m, k), (b, m), (m, k), (b, d), (1,)])
    for turn in range(2):
        d_W = gu.dev(W)
        m1.zero_(), m2.zero_()
        L.train_step(d_x, d_idx, d_W, m1, m2, d_off, d_lab, 1, scale, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
        ref_loss, ref_g = orc.sqh_loss_grad(orc.forward(x, idx, W), off, lab, scale)
        got_g = gu.host(g)
        assert_close(got_g, ref_g, 1e-5, "g")
        share = (got_g != 0).mean(axis=1)
        assert (share.max() > 1 / 32) == crowded and share.min() < 1 / 32
        assert abs(float(loss) - ref_loss) <= 1e-5 * abs(ref_loss)
        assert_close(gu.host(gW), orc.backward_weight(got_g, x, idx), 1e-5, "grad_W")
        assert_close(gu.host(gx), orc.backward_input(got_g, idx, W, d), 1e-4, "grad_x")
    L.close()


@pytest.mark.parametrize("m,b", [(200031, 5), (98304, 3), (65537, 40)])
def test_lists_of_several_workgroups(orc, m, b, monkeypatch):
    """A list is written by a workgroup for every 32 768 labels: nearly all of its entries from one of them, thousands of it, up to what the list holds; a last
    workgroup of one word; instances with none and with a single nonzero in the last label."""
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SPARSE", "always")
    print("lists of several workgroups", m, b, flush=True)
    d, k = 64, 8
    cfg = wl.custom(m, d, k, b, positives=3, index=996)
    idx = wl.gen_idx(cfg)
    x = np.ones((b, d), np.float32)
    x[1] *= 1e3
    W = np.full((m, k), -1.0, np.float32)
    W[7: 7 + m // 32 - 60] = np.float32(-0.05)     # inside the margin, but for instance 1
    W[m // 2: m // 2 + 3] = np.float32(-0.01)
    off, lab = np.arange(b + 1, dtype=np.int64), np.full(b, m - 1, np.int32)
    L = usl.Layer(m, d, k, b)
    m1, m2, g, gW, gx, loss = (gu.empty(s).fill_(float("nan")) for s in [(m, k), (m, k), (b, m), (m, k), (b, d), (1,)])
    for turn in range(3):
        m1.zero_(), m2.zero_()
        L.train_step(gu.dev(x), gu.dev(idx), gu.dev(W), m1, m2, gu.dev(off), gu.dev(lab), 1, 1.0, 1, 0.0, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
        L.invalidate()
        ref_loss, ref_g = orc.sqh_loss_grad(orc.forward(x, idx, W), off, lab, 1.0)
        got_g = gu.host(g)
        assert_close(got_g, ref_g, 1e-5, "g")
        count = (got_g != 0).sum(axis=1)
        assert count[1] == 1 and m // 32 - 60 < count[0] <= m // 32
        assert abs(float(loss) - ref_loss) <= 1e-5 * abs(ref_loss)
        assert_close(gu.host(gW), orc.backward_weight(got_g, x, idx), 1e-5, "grad_W")
        assert_close(gu.host(gx), orc.backward_input(got_g, idx, W, d), 1e-4, "grad_x")
    L.close()
