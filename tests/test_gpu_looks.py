"""Looks at the gradient (csrc/k_sparse_grad.hip) one after another on one context: each starts from the word that the one before
left, whatever that one found, with other batches, and with rows longer than one turn of the sample's loads (1 048 576 labels)."""
import pytest

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k,max_b", [(65536, 3, 300), (1048576 + 3, 1, 5), (1048576 + 1028, 2, 2)])
def test_looks_in_turn(orc, monkeypatch, m, k, max_b):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SPARSE", "always")
    d = 40
    cfg = wl.custom(m, d, k, max_b, positives=3, index=910 + max_b)
    idx, W, x, g = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg), wl.gen_g(cfg)
    sparse, one_full = g.copy(), g.copy()
    sparse[wl.rng(cfg, 21).random(g.shape) < 0.999] = 0.0
    one_full[:] = sparse
    one_full[-1, :m // 16] = g[-1, :m // 16]   # twice what its list holds
    L = usl.Layer(m, d, k, max_b)
    d_idx, d_W, d_x = gu.dev(idx), gu.dev(W), gu.dev(x)
    for name, of, b in (("sparse", sparse, max_b), ("dense", g, max_b), ("sparse", sparse, max_b - 1), ("one full", one_full, max_b), ("sparse", sparse, max_b)):
        print("look", m, name, b, flush=True)
        d_g = gu.dev(of[:b])
        gW, gx = gu.empty((m, k)).fill_(float("nan")), gu.empty((b, d)).fill_(float("nan"))
        L.backward_weight(d_g, d_x[:b], d_idx, gW, b)
        L.backward_input(d_g, d_idx, d_W, gx, b)
        assert_close(gu.host(gW), orc.backward_weight(of[:b], x[:b], idx), 1e-5, "grad_W")
        assert_close(gu.host(gx), orc.backward_input(of[:b], idx, W, d), 1e-4, "grad_x")
    L.close()
