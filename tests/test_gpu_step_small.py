"""usl_train_step of small layers (k_step_small.hip: the whole step in two launches) against the oracle, where it can go wrong: a
last workgroup of few labels, fan-ins beside the kernel's own, batches that are no multiple of four, four and eight wavefronts, long rows of few instances, features
without a connection, targets listed twice or outside the layer, and an order of the connections that is none (new scratch, and idx
replaced behind the library's back).  The general path runs on the same inputs."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu

# (m, d, k, b, storage, loss_kind)
CASES = [(1, 1, 1, 1, "f32", 0), (63, 40, 7, 3, "f32", 1), (64, 8, 8, 4, "bf16", 0), (65, 33, 9, 5, "f32", 0), (130, 16, 16, 33, "bf16", 1),
         (129, 64, 31, 32, "f32", 0), (1024, 64, 8, 16, "f32", 1), (1000, 700, 32, 18, "f32", 0), (640, 32, 32, 100, "bf16", 0),
         (2111, 1500, 3, 9, "f32", 1), (300, 50, 17, 201, "f32", 0), (4100, 90, 5, 40, "bf16", 1), (20000, 128, 16, 8, "f32", 0),
         (300, 700, 8, 3, "f32", 0), (130, 200, 16, 8, "bf16", 1), (200, 1001, 20, 5, "f32", 1), (70, 129, 3, 1, "f32", 0)]   # columns shared by wavefronts


@pytest.mark.parametrize("path", ["small", "general"])
@pytest.mark.parametrize("m,d,k,b,storage,loss_kind", CASES)
def test_steps_of_a_small_layer(orc, m, d, k, b, storage, loss_kind, path, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SMALL", "on" if path == "small" else "off")
    print("small step", m, d, k, b, storage, loss_kind, path, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=min(3, m), index=900 + CASES.index((m, d, k, b, storage, loss_kind)))
    hp = wl.ADAM
    W, x = wl.gen_W(cfg), wl.gen_x(cfg)
    off, lab = wl.gen_targets(cfg)
    lists = [list(lab[off[i]:off[i + 1]]) for i in range(b)]
    lists[0] = lists[0] + lists[0][:1]                       # a label twice
    if b > 2:
        lists[1], lists[2] = [], list(range(0, m, 2))        # none, many
    lists[b - 1] = [m - 1, 0]
    off = np.cumsum([0] + [len(l) for l in lists]).astype(np.int64)
    lab = np.array([v for l in lists for v in l], np.int32)
    r = wl.rng(cfg, 5)
    m1, m2 = (r.standard_normal((m, k)) * 1e-3).astype(np.float32), (r.random((m, k)) * 1e-6).astype(np.float32)
    scale = float(np.float32(1.0 / b))
    L = usl.Layer(m, d, k, b, storage)
    d_idx = gu.dev(wl.gen_idx(cfg))
    d_W, d_x, d_m1, d_m2, d_off, d_lab = gu.dev(W), gu.dev(x), gu.dev(m1), gu.dev(m2), gu.dev(off), gu.dev(lab)
    g, gW, gx, loss = gu.empty((b, m)), gu.empty((m, k)), gu.empty((b, d)), gu.empty((1,))
    for t in range(1, 5):
        if t == 3:
            L.redistribute(d_idx, d_W, d_m1, d_m2, 0.3, 11, t)
        if t == 4 and path == "small":   # other connections at the same address, without a word
            other = torch.from_numpy(wl.gen_idx(wl.custom(m, d, k, b, index=950))).cuda()
            d_idx.data.view(-1)[:] = other.view(-1)
        idx, W, m1, m2 = gu.host(d_idx).copy(), gu.host(d_W).copy(), gu.host(d_m1).copy(), gu.host(d_m2).copy()
        for out in (g, gW, gx):
            out.fill_(float("nan"))
        want_gx = t != 2
        L.train_step(d_x, d_idx, d_W, d_m1, d_m2, d_off, d_lab, loss_kind, scale, t, hp["lr"], hp["beta1"], hp["beta2"], hp["eps"],
                     g, gW, gx if want_gx else None, loss, b)
        ref_loss, ref_g = (orc.bce_loss_grad if loss_kind == 0 else orc.sqh_loss_grad)(orc.forward(x, idx, W), off, lab, scale)
        got_g, got_gW = gu.host(g), gu.host(gW)
        assert_close(got_g, ref_g, 1e-5, "g")
        assert abs(float(loss.item()) - ref_loss) <= 1e-5 * abs(ref_loss)
        assert_close(got_gW, orc.backward_weight(got_g, x, idx), 1e-5, "grad_W")
        if want_gx:
            assert_close(gu.host(gx), orc.backward_input(got_g, idx, W, d), 1e-4, "grad_x")
            again = gu.host(gx).copy()
            L2, W2 = usl.Layer(m, d, k, b, storage), gu.dev(W)   # new scratch: the same bits, whatever it held
            L2.train_step(d_x, d_idx, W2, gu.dev(m1), gu.dev(m2), d_off, d_lab, loss_kind, scale, t, hp["lr"], hp["beta1"], hp["beta2"],
                          hp["eps"], g, gW, gx, loss, b)
            if path == "small":
                np.testing.assert_array_equal(gu.host(gx), again)
            L2.close()
        pre = orc.adam_step(W, got_gW, m1, m2, t, hp["lr"], hp["beta1"], hp["beta2"], hp["eps"])
        assert_close(gu.host(d_m1), m1, 1e-4, "m1")
        assert_close(gu.host(d_m2), m2, 1e-4, "m2")
        if storage == "f32":
            assert_close(gu.host(d_W), W, 1e-4, "W")
        else:   # rounded to bfloat16: see test_gpu_parity.test_adam
            got = wl.as_f32(gu.host(d_W)).astype(np.float64)
            ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(pre), 1e-30))) - 7)
            rms = float(np.sqrt(np.mean(pre.astype(np.float64) ** 2)))
            assert (np.abs(got - pre) <= 0.5 * ulp * (1 + 1e-3) + 1e-4 * np.abs(pre) + 1e-4 * rms).all()
    L.close()


def test_targets_outside_the_layer_and_infinite_activations():
    """A label that does not exist is no target; an infinite activation reaches only what is connected to it."""
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    m, d, k, b = 100, 30, 4, 6
    gen = torch.Generator().manual_seed(3)
    idx = torch.stack([torch.randperm(d - 1, generator=gen)[:k] for _ in range(m)]).to(torch.int32)   # nobody has feature d - 1 ...
    idx[7, 2] = d - 1                                                                                # ... but label 7
    x = torch.rand((b, d), generator=gen)
    x[4, d - 1] = float("inf")
    W = torch.rand((m, k), generator=gen) + 0.1
    res = {}
    for bad in (False, True):
        lab = torch.tensor([1, 2, -5 if bad else 3, m if bad else 3, 3, 99], dtype=torch.int32)
        off = torch.tensor([0, 1, 5, 5, 5, 5, 6], dtype=torch.int64)
        L = usl.Layer(m, d, k, b)
        g, gW, gx, loss = gu.empty((b, m)), gu.empty((m, k)), gu.empty((b, d)), gu.empty((1,))
        zeros = lambda: torch.zeros((m, k), device="cuda")
        L.train_step(x.cuda(), idx.cuda(), W.cuda(), zeros(), zeros(), off.cuda(), lab.cuda(), 0, 1.0, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
        res[bad] = (g.cpu(), gW.cpu(), gx.cpu())
        L.close()
    for u, v in zip(res[False], res[True]):
        assert torch.equal(torch.nan_to_num(u), torch.nan_to_num(v))
    g, gW, gx = res[False]
    assert torch.isfinite(g).all() and float(g[4, 7]) == 1.0      # sigmoid of an infinite score
    others = torch.ones(m, dtype=torch.bool)
    others[7] = False
    assert torch.isfinite(gW[others]).all() and not torch.isfinite(gW[7, 2])
    assert torch.isfinite(gx).all()
