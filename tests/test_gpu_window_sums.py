"""The sums of the input gradient's windows (k_lf_reduce): few lanes add eight or four windows at a time, many one by one.  Weights and
gradients are small whole numbers, so every sum is exact in float32 whatever its order, and the result is compared for equality."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# rows of 8192 features: 32 of them are the most for which eight windows' loads go out together on 256 compute units, 64 for four
@pytest.mark.parametrize("b", [1, 32, 33, 64, 65])
@pytest.mark.parametrize("m,d,k", [(60000, 8192, 16), (40001, 8190, 9)])   # ... and rows that are padded
def test_sums_of_windows(m, d, k, b):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    print("window sums", m, d, k, b, flush=True)
    rng = np.random.default_rng(m + b)
    idx = ((rng.integers(0, d, (m, 1)) + np.arange(k) * (d // k)) % d).astype(np.int32)
    W = rng.integers(-4, 5, (m, k)).astype(np.float32)
    g = rng.integers(-4, 5, (b, m)).astype(np.float32)
    x = rng.integers(-2, 3, (b, d)).astype(np.float32)
    L = usl.Layer(m, d, k, b)
    d_g, d_idx, d_W = gu.dev(g), gu.dev(idx), gu.dev(W)
    gW, gx = gu.empty((m, k)).fill_(float("nan")), gu.empty((b, d)).fill_(float("nan"))
    L.backward(d_g, gu.dev(x), d_idx, d_W, gW, gx, b)
    flat = idx.ravel()
    want = np.stack([np.bincount(flat, weights=(W * g[i][:, None]).ravel(), minlength=d) for i in range(b)])
    assert np.abs(want).max() < 2 ** 24
    np.testing.assert_array_equal(gu.host(gx), want.astype(np.float32))
    i = b - 1
    if b == 1:
        np.testing.assert_array_equal(gu.host(gW), g[i][:, None] * x[i][idx])
    L.check()
    L.close()
