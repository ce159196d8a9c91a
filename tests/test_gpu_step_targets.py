"""The targets inside forward, in usl_train_step: every instance has targets in the first and the last lane of a wavefront and of the layer, in
all of a wavefront and in none; instance 31 and 32 lie in different words of marks.  And the fingerprint of idx that is compared beside
them: other contents in any one of its 64 parts are noticed."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


# layouts of one, two and four instances a read, rows in two halves, blocks of equal size, with and without a copy of x
@pytest.mark.parametrize("loss_kind", [0, 1])
@pytest.mark.parametrize("m,d,k,b,storage", [(20011, 600, 32, 35, "f32"), (9001, 12000, 32, 34, "f32"), (5003, 32768, 32, 33, "f32"),
                                             (3001, 41000, 8, 34, "f32"), (20011, 8192, 24, 66, "bf16"), (5003, 65536, 32, 33, "bf16")])
def test_gradient_of_targets_and_others(m, d, k, b, storage, loss_kind, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SMALL", "off")
    print("targets", m, d, k, b, storage, loss_kind, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=990)
    d_idx, W, d_x = gu.dev(wl.gen_idx(cfg)), wl.gen_W(cfg), gu.dev(wl.gen_x(cfg))
    scale = float(np.float32(1.0 / b))
    L = usl.Layer(m, d, k, b, storage)
    for turn in range(2):   # the second turn's targets are others: no mark of the first may be left
        lists = [[0, 63, 64, 1023, 1024, m - 1, m // 2 + 7 * i + turn] for i in range(b)]
        lists[3 + turn], lists[5] = [], list(range(64 * turn, 64 * turn + 64))
        lists[31], lists[32] = [5 + turn, 5 + turn], [6, 2047, 2048 + turn]
        off = gu.dev(np.cumsum([0] + [len(q) for q in lists]).astype(np.int64))
        lab = gu.dev(np.concatenate([np.asarray(q, dtype=np.int32) for q in lists]))
        d_W = gu.dev(W)
        ref, ref_loss = gu.empty((b, m)), gu.empty((1,))
        L.forward(d_x, d_idx, d_W, ref, b)
        (L.bce_loss_grad if loss_kind == 0 else L.sqh_loss_grad)(ref, off, lab, scale, ref, ref_loss, b)
        m1, m2 = gu.empty((m, k)).fill_(0.0), gu.empty((m, k)).fill_(0.0)
        g, gW, gx, loss = gu.empty((b, m)), gu.empty((m, k)), gu.empty((b, d)), gu.empty((1,)).fill_(float("nan"))
        L.train_step(d_x, d_idx, d_W, m1, m2, off, lab, loss_kind, scale, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
        assert torch.equal(g, ref)
        # both are float32 sums of a few losses at a time, added up in float64
        assert abs(float(loss) - float(ref_loss)) <= 1e-6 * abs(float(ref_loss))
    L.close()


@pytest.mark.parametrize("m,d,k", [(70001, 3000, 12), (500, 40, 7)])
def test_other_connections_in_one_part_are_noticed(m, d, k, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SMALL", "off")
    b = 8
    print("part of idx", m, d, k, flush=True)
    cfg = wl.custom(m, d, k, b, positives=3, index=991)
    d_idx, d_W, d_x = gu.dev(wl.gen_idx(cfg)), gu.dev(wl.gen_W(cfg)), gu.dev(wl.gen_x(cfg))
    off, lab = (gu.dev(a) for a in wl.gen_targets(cfg))
    m1, m2, g, gW, gx, loss = (gu.empty(s).fill_(0.0) for s in [(m, k), (m, k), (b, m), (m, k), (b, d), (1,)])
    step = lambda L: L.train_step(d_x, d_idx, d_W, m1, m2, off, lab, 0, 1.0 / b, 1, 0.0, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
    groups = m * k // 4
    samples = min(groups, 4096)
    parts = (samples + 63) // 64
    for part in (0, parts // 2, parts - 1, None):   # None: the values behind the last whole group of four
        if part is None and m * k % 4 == 0:
            continue
        at = m * k - 1 if part is None else part * 64 * (groups // samples) * 4
        L = usl.Layer(m, d, k, b)
        step(L)
        step(L)
        L.check()
        assert not torch.isnan(gx).any()
        flat = d_idx.data.view(-1)
        flat[at] = (int(flat[at]) + 1) % d    # (`.data`: without the binding's notice)
        step(L)
        with pytest.raises(Exception):
            L.check()
        assert torch.isnan(gx).all()
        L.close()
