"""usl_train_step's loss inside the forward kernel, where it can go wrong: labels listed twice, instances without targets,
padded fan-ins, every layout of the activations, rows in two halves, targets of one label in every instance.  The
gradient has to equal that of the separate calls bit for bit, the loss the oracle's."""
import numpy as np
import pytest

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu


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
