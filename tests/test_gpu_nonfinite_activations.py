"""An activation that is infinite or NaN reaches the labels that are connected to it and no others, also where the fan-in
is padded: what the slots that do not exist read is no real column.  Every layout of the activations, against the oracle:
the same NaNs and infinities, everything else as close as ever."""
import numpy as np
import pytest

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu

# (m, d, k, b, storage)
SHAPES = [
    (3001, 300, 24, 1, "f32"), (3001, 300, 5, 1, "bf16"), (3001, 304, 47, 2, "bf16"), (3001, 300, 48, 4, "f32"),   # streamed: 4 * LPL slots
    (3001, 300, 12, 9, "f32"), (3001, 12000, 33, 6, "f32"), (3001, 24000, 7, 5, "bf16"),                          # units of 4 and 2
    (3001, 41000, 12, 5, "f32"), (3001, 65535, 5, 3, "f32"), (3001, 65532, 63, 2, "f32"), (3001, 65535, 20, 5, "bf16"),   # two halves, one unit
    (3001, 65536, 20, 5, "f32"), (3001, 65536, 33, 1, "f32"), (3001, 65536, 20, 70, "bf16"), (3001, 65536, 20, 1, "bf16"),   # no room for a column of zeros
]


def same(a, r):
    np.testing.assert_array_equal(np.isnan(a), np.isnan(r))
    np.testing.assert_array_equal(np.where(np.isinf(r), r, 0), np.where(np.isinf(a), a, 0))
    fine = np.isfinite(r)
    assert fine.any() and not fine.all()
    assert_close(a[fine], r[fine], 1e-5, "finite scores")


# small: layers that have a step of their own (fewer slots than 32 and short rows, or few instances), which the general path takes too
@pytest.mark.parametrize("m,d,k,b,storage,small", [s + ("off",) for s in SHAPES] + [s + ("on",) for s in SHAPES if s[1] < 1000 and s[2] <= 32])
def test_nonfinite_activations_stay_with_their_labels(orc, m, d, k, b, storage, small, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_SMALL", small)
    print("nonfinite activations", m, d, k, b, storage, small, flush=True)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=840 + SHAPES.index((m, d, k, b, storage)))
    idx, W, x = wl.gen_idx(cfg), wl.gen_W(cfg), wl.as_f32(wl.gen_x(cfg)).copy()
    x[0, 0], x[0, d - 1], x[b - 1, 7] = np.inf, -np.inf, np.nan
    if b > 64:
        x[65, 0] = np.nan
    x = wl.store(x, storage)
    for j in range(20):   # a few labels that do have a connection to them, whatever was drawn
        rest = [c for c in idx[j].tolist() if c not in (0, 7, d - 1)]
        idx[j] = ([(0, 7, d - 1)[j % 3]] + rest + [c for c in range(8, 200) if c not in rest])[:k]
    d_idx, d_W, d_x, out = gu.dev(idx), gu.dev(W), gu.dev(x), gu.empty((b, m)).fill_(1.0)
    L = usl.Layer(m, d, k, b, storage)
    L.forward(d_x, d_idx, d_W, out, b)
    same(gu.host(out), orc.forward(x, idx, W))
    # the training step computes the same scores on its way to the gradient
    off, lab = np.arange(b + 1, dtype=np.int64), np.zeros(b, dtype=np.int32)
    d_off, d_lab, loss = gu.dev(off), gu.dev(lab), gu.empty((1,))
    L.bce_loss_grad(out, d_off, d_lab, 1.0, out, loss, b)
    g, gW, m1, m2 = gu.empty((b, m)), gu.empty((m, k)), gu.empty((m, k)).fill_(0.0), gu.empty((m, k)).fill_(0.0)
    L.train_step(d_x, d_idx, d_W, m1, m2, d_off, d_lab, 0, 1.0, 1, 1e-3, 0.9, 0.999, 1e-8, g, gW, None, loss, b)
    np.testing.assert_array_equal(gu.host(g), gu.host(out))
    L.close()
