"""The per-instance lists of nonzero gradients (csrc/k_sparse_grad.hip): the counts are cleared for every instance, also where a
batch has more of them than the clearing kernel has lanes, and call by call where batches shrink and grow."""
import pytest

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_b,batches", [(1, (1, 1)), (257, (256, 257, 3, 257)), (600, (600, 31, 32, 600))])
def test_counts_are_cleared_for_every_instance(orc, monkeypatch, max_b, batches):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SPARSE", "always")
    m, d, k = 65536, 40, 3
    cfg = wl.custom(m, d, k, max_b, positives=3, index=880 + max_b)
    idx, W, x, g = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg), wl.gen_g(cfg)
    g[wl.rng(cfg, 21).random(g.shape) < 0.999] = 0.0
    L = usl.Layer(m, d, k, max_b)
    d_idx, d_W, d_x, d_g = gu.dev(idx), gu.dev(W), gu.dev(x), gu.dev(g)
    for b in batches:
        print("counts", max_b, b, flush=True)
        gW, gx = gu.empty((m, k)).fill_(float("nan")), gu.empty((b, d)).fill_(float("nan"))
        L.backward_weight(d_g[:b], d_x[:b], d_idx, gW, b)
        L.backward_input(d_g[:b], d_idx, d_W, gx, b)
        assert_close(gu.host(gW), orc.backward_weight(g[:b], x[:b], idx), 1e-5, "grad_W")
        assert_close(gu.host(gx), orc.backward_input(g[:b], idx, W, d), 1e-4, "grad_x")
    L.close()
