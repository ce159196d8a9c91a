"""usl_backward_input and usl_backward have private lists of their own, side by side: alternating them builds nothing
anew, and a changed idx is noticed by each (a rebuild would go unnoticed: it would give the new contents' numbers)."""
import numpy as np
import pytest
import torch

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form", ["l2", "lds"])
@pytest.mark.parametrize("other_first", [False, True])
def test_lists_of_both_entry_points_are_kept(orc, form, other_first, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_BOTH", "on")
    monkeypatch.setenv("USL_TUNE_BWI", form)
    m, d, k, b = 70000, 2048, 2, 4
    cfg = wl.custom(m, d, k, b, positives=3, index=870)
    idx, W, x, g = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg), wl.gen_g(cfg)
    L = usl.Layer(m, d, k, b)
    d_idx, d_W, d_x, d_g = gu.dev(idx), gu.dev(W), gu.dev(x), gu.dev(g)
    gW, gx = gu.empty((m, k)), gu.empty((b, d))
    p = lambda t: t.data_ptr()   # addresses: the binding's own look at the tensor is left out
    one = lambda: L.backward_input(p(d_g), p(d_idx), p(d_W), p(gx), b)
    both = lambda: L.backward(p(d_g), p(d_x), p(d_idx), p(d_W), p(gW), p(gx), b)
    first, second = (both, one) if other_first else (one, both)
    for call in (first, second, first, second):
        gx.fill_(7.0)
        call()
        assert_close(gu.host(gx), orc.backward_input(g, idx, W, d), 1e-4, "grad_x")
    L.check()
    d_idx.copy_(torch.from_numpy(wl.gen_idx(wl.custom(m, d, k, b, index=871))))
    for call in (first, second):   # both sets of lists stand, and both are of the old contents
        call()
        assert torch.isnan(gx).all()
        with pytest.raises(usl.UslError) as e:
            L.check()              # drops all lists
        assert e.value.status == usl.USL_ESTALE
        d_idx.copy_(torch.from_numpy(idx))
        for again in (first, second):
            again()
            assert np.isfinite(gu.host(gx)).all()
        L.check()
        d_idx.copy_(torch.from_numpy(wl.gen_idx(wl.custom(m, d, k, b, index=871))))
    L.close()
