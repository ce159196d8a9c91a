"""Redistribution where most magnitudes equal the threshold: those that go are the first in flat order, counted over several
workgroups of 4096 values and the lanes' pieces of 16 bytes.  And rows whose first candidates clash.  Bit for bit against the
oracle."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,d,k,storage,frac,few", [(3001, 400, 5, "f32", 0.37, 0.02), (3001, 400, 5, "bf16", 0.37, 0.02), (4096, 64, 3, "f32", 0.5, 0.0),
                                                    (4099, 64, 3, "bf16", 0.9, 0.3), (1021, 40, 33, "f32", 0.25, 0.1), (2000, 70, 64, "bf16", 0.3, 0.1),
                                                    (70001, 40, 31, "f32", 0.1, 0.5)])
def test_ties_over_many_workgroups(orc, m, d, k, storage, frac, few):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    print("redistribute", m, d, k, storage, frac, few, flush=True)
    rng = np.random.default_rng(m + k)
    idx = np.argsort(rng.random((m, d)), axis=1)[:, :k].astype(np.int32)
    Wf = np.where(rng.random((m, k)) < 0.5, 0.5, -0.5).astype(np.float32)
    other = rng.random((m, k)) < few      # some below and some above the others
    Wf[other] = rng.standard_normal(int(other.sum())).astype(np.float32)
    W = wl.store(Wf, storage)
    m1, m2 = rng.standard_normal((m, k)).astype(np.float32), rng.random((m, k)).astype(np.float32)
    L = usl.Layer(m, d, k, 1, storage)
    d_idx, d_W, d_m1, d_m2 = gu.dev(idx), gu.dev(W), gu.dev(m1), gu.dev(m2)
    n = L.redistribute(d_idx, d_W, d_m1, d_m2, frac, 77, 2)
    n_ref, _ = orc.redistribute(idx, W, m1, m2, d, frac, 77, 2)     # in place on the host copies
    assert n == n_ref
    np.testing.assert_array_equal(gu.host(d_W).view(np.uint8), W.view(np.uint8))
    np.testing.assert_array_equal(gu.host(d_m1), m1)
    np.testing.assert_array_equal(gu.host(d_m2), m2)
    np.testing.assert_array_equal(gu.host(d_idx), idx)
    assert L.validate_indices(d_idx) == 0
    L.close()


# 2^25 lanes (32, 64, 8 to a row) and a few: the smallest layers with eight turns of rows to a wavefront on 256 compute units; just below;
# as large, but narrow: slots clash, one turn.  In the first two every other row of new slots clashes, too.
@pytest.mark.parametrize("m,d,k,per_row", [(1048577, 512, 31, 2), (524289, 1024, 64, 3), (4194304, 160, 5, 1), (1048575, 512, 32, 1), (1048580, 100, 32, 1)])
def test_turns_of_rows_in_large_layers(orc, m, d, k, per_row):
    import torch
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    print("turns", m, d, k, per_row, flush=True)
    L = usl.Layer(m, d, k, 1)
    d_idx = gu.empty((m, k), torch.int32).fill_(-7)
    L.init_indices(d_idx, 0xABCDEF)
    idx = orc.init_indices(m, d, k, 0xABCDEF)
    np.testing.assert_array_equal(gu.host(d_idx), idx)
    W = np.random.default_rng(m).standard_normal((m, k), dtype=np.float32)
    W[::3] = 1.0      # ties
    m1, m2 = W * np.float32(0.5), np.abs(W)
    d_W, d_m1, d_m2 = gu.dev(W), gu.dev(m1), gu.dev(m2)
    L.redistribute_rows(d_idx, d_W, d_m1, d_m2, per_row, 77, 2)
    orc.redistribute_rows(idx, W, m1, m2, d, per_row, 77, 2)     # in place on the host copies
    np.testing.assert_array_equal(gu.host(d_idx), idx)
    np.testing.assert_array_equal(gu.host(d_W).view(np.uint8), W.view(np.uint8))
    assert L.validate_indices(d_idx) == 0
    L.close()
