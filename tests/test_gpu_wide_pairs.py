"""Forward of wide bfloat16 rows with fan-ins of 49 to 64 as 1024 lanes with one label each: last workgroups of few labels, padded fan-ins, two
instances a read and one, with the loss and with marked nonzeros."""
import numpy as np
import pytest

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,k,b", [(1025, 21000, 64, 5), (3000, 40000, 50, 34), (2047, 45000, 64, 3), (1100, 65536, 64, 4), (1030, 65536, 57, 3), (66000, 25000, 49, 5)])
def test_one_label_a_lane(orc, m, d, k, b, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SHAPE", "3")
    monkeypatch.setenv("USL_TUNE_SPARSE", "always")
    print("wide pairs", m, d, k, b, flush=True)
    cfg = wl.custom(m, d, k, b, storage="bf16", positives=3, index=997)
    idx, W, x = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg)
    off, lab = wl.gen_targets(cfg)
    L = usl.Layer(m, d, k, b, "bf16")
    d_idx, d_x, out = gu.dev(idx), gu.dev(x), gu.empty((b, m))
    ref = orc.forward(x, idx, W)
    L.forward(d_x, d_idx, gu.dev(W), out, b)
    assert_close(gu.host(out), ref, 1e-5, "out")
    scale = float(np.float32(1.0 / b))
    for loss_kind in (0, 1):
        ref_loss, ref_g = (orc.bce_loss_grad if loss_kind == 0 else orc.sqh_loss_grad)(ref, off, lab, scale)
        m1, m2, g, gW, gx, loss = (gu.empty(s).fill_(0.0) for s in [(m, k), (m, k), (b, m), (m, k), (b, d), (1,)])
        L.train_step(d_x, d_idx, gu.dev(W), m1, m2, gu.dev(off), gu.dev(lab), loss_kind, scale, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, gx, loss, b)
        assert_close(gu.host(g), ref_g, 1e-5, "g")
        assert abs(float(loss) - ref_loss) <= 1e-5 * abs(ref_loss)
        assert_close(gu.host(gW), orc.backward_weight(gu.host(g), x, idx), 1e-5, "grad_W")
    L.close()
