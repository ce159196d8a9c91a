"""The scratch of a layer is sized by its first calls for every batch up to max_b: a later call, with whatever batch,
allocates nothing (growing a buffer waits for the stream in the middle of training).  Watched through the device's free
memory, around layers whose batches are split into more parts when they are smaller."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,k,max_b,first", [(13330, 5000, 32, 128, 128), (13330, 5000, 32, 128, 6), (30938, 1024, 32, 300, 300),
                                               (60000, 40000, 16, 100, 33), (250000, 600, 8, 70, 70)])
def test_no_later_batch_grows_the_scratch(m, d, k, max_b, first):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    print("scratch", m, d, k, max_b, first, flush=True)
    cfg = wl.custom(m, d, k, max_b, positives=3, index=860)
    idx, W, x, g_in = gu.dev(wl.gen_idx(cfg)), gu.dev(wl.gen_W(cfg)), gu.dev(wl.gen_x(cfg)), gu.dev(wl.gen_g(cfg))
    m1, m2 = gu.empty((m, k)).fill_(0.0), gu.empty((m, k)).fill_(0.0)
    off, lab = gu.dev(np.arange(max_b + 1, dtype=np.int64)), gu.dev(np.arange(max_b, dtype=np.int32))
    g, gW, gx, loss = gu.empty((max_b, m)), gu.empty((m, k)), gu.empty((max_b, d)), gu.empty((1,))

    def calls(L, b):
        L.train_step(x, idx, W, m1, m2, off, lab, 0, 1.0 / b, 1, 0.0, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
        L.forward(x, idx, W, g, b)
        L.bce_loss_grad(g, off, lab, 1.0 / b, g, loss, b)
        L.backward(g_in, x, idx, W, gW, gx, b)
        L.backward_weight(g_in, x, idx, gW, b)
        L.backward_input(g_in, idx, W, gx, b)
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    batches = [max_b, max_b - 1, max_b * 3 // 4, max_b // 2, 48, 32, 17, 8, 6, 5, 4, 3, 2, 1, max_b]
    L = usl.Layer(m, d, k, max_b)   # the runtime loads a kernel's code, which takes memory too, when it is first launched
    for b in batches:
        calls(L, b)
    L.close()
    L = usl.Layer(m, d, k, max_b)
    free = calls(L, first)
    for b in batches:
        assert calls(L, b) == free, "a batch of %d after one of %d" % (b, first)
    L.close()


def test_parts_asked_for_by_hand_between_calls(orc, monkeypatch):
    """The tuning aids are read on every call: scratch that was sized under one setting has to serve the next."""
    import gpu_util as gu
    from helpers import assert_close
    from paper_2306_03725_amd import usl
    m, d, k, b = 13330, 5000, 32, 96
    cfg = wl.custom(m, d, k, b, positives=3, index=865)
    h_idx, h_W, h_x, h_g = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg), wl.gen_g(cfg)
    idx, W, x, g = gu.dev(h_idx), gu.dev(h_W), gu.dev(h_x), gu.dev(h_g)
    gW, gx = gu.empty((m, k)), gu.empty((b, d))
    L = usl.Layer(m, d, k, b)
    for parts in ("1", None, "3", "24", None):
        if parts:
            monkeypatch.setenv("USL_TUNE_BOTH_PARTS", parts)
        else:
            monkeypatch.delenv("USL_TUNE_BOTH_PARTS", raising=False)
        gW.fill_(7.0); gx.fill_(7.0)
        L.backward(g, x, idx, W, gW, gx, b)
        assert_close(gu.host(gW), orc.backward_weight(h_g, h_x, h_idx), 1e-5, "grad_W")
        assert_close(gu.host(gx), orc.backward_input(h_g, h_idx, h_W, d), 1e-4, "grad_x")
    L.close()
