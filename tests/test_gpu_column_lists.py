"""The lists of usl_backward_input's form over L2 (count, order, fill).  Weights and gradients are small whole numbers, so
that every sum is exact in float32 whatever its order: a connection that is missing, listed twice or put into another
feature's list shows, and the result is compared for equality."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (m, d, k, labels of a window, which features the connections reach)
CASES = [
    (1, 1, 1, 0, "all"),
    (5000, 1, 1, 0, "all"),             # one list of 5000 entries, beyond the last bucket
    (3001, 1023, 5, 0, "all"),          # around one chunk of 1024 features
    (3001, 1024, 5, 0, "all"),
    (3001, 1025, 5, 0, "all"),
    (20011, 3075, 7, 0, "few"),         # long lists in one chunk, empty ones in the others; shares with ragged ends
    (20011, 3075, 7, 0, "last"),        # the first chunks empty
    (9973, 5000, 9, 611, "all"),        # windows that begin off every alignment
    (9973, 4096, 3, 13, "all"),         # 768 windows: chunks of 4096 features
    (9973, 4097, 3, 13, "all"),         # ... and one feature
    (40000, 9000, 2, 64, "few"),
]


@pytest.mark.parametrize("m,d,k,win,reach", CASES)
def test_sums_over_the_column_lists(m, d, k, win, reach, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_BWI", "l2")
    if win:
        monkeypatch.setenv("USL_TUNE_WIN", str(win))
    print("column lists", m, d, k, win, reach, flush=True)
    b = 3
    rng = np.random.default_rng(m + d)
    width = d if reach == "all" else max(k, 11)
    first = d - width if reach == "last" else 0
    idx = np.argsort(rng.random((m, min(width, 64))), axis=1)[:, :k] if width <= 64 else \
        (rng.integers(0, d, (m, 1)) + np.arange(k) * (d // k)) % d
    idx = (idx + first).astype(np.int32)
    W = rng.integers(-8, 9, (m, k)).astype(np.float32)
    g = rng.integers(-8, 9, (b, m)).astype(np.float32)
    L = usl.Layer(m, d, k, b)
    gx = gu.empty((b, d)).fill_(float("nan"))
    L.backward_input(gu.dev(g), gu.dev(idx), gu.dev(W), gx, b)
    want = np.zeros((b, d), np.int64)
    for i in range(b):
        np.add.at(want[i], idx.ravel(), (W * g[i][:, None]).astype(np.int64).ravel())
    assert np.abs(want).max() < 2 ** 24
    np.testing.assert_array_equal(gu.host(gx).astype(np.int64), want)
    L.check()
    L.close()
