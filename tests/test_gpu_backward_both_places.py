"""Where k_both_lds takes its weights from and leaves its weight gradients: places of 16 bits for a workgroup whose
connections LDS holds at a time, one by one for the others (a skewed connectivity), and added to where the batch goes
through in several passes.  Against the oracle, element by element."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_backward_both import run_and_compare

pytestmark = pytest.mark.gpu

# (m, d, k, b, storage, connections: of the first block of features only; of all)
CASES = [
    (40000, 4096, 4, 5, "bf16", "one block"),     # two instances at a time, about 64000 connections to a workgroup
    (20000, 8192, 32, 6, "f32", "one block"),     # four at a time, about 130000
    (20000, 8192, 32, 3, "bf16", "one block"),
    (9001, 4099, 7, 301, "f32", "one block"),     # three passes over the batch
    (9001, 4099, 7, 301, "bf16", "all"),
    (513, 2048, 16, 5, "f32", "all"),             # fewer than eight connections to a lane
    (521, 2048, 16, 5, "f32", "all"),             # ... just more
    (40001, 2047, 3, 4, "bf16", "all"),           # one block: places are flat slots
    # around four at a time with the activations in the place of the sums (windows of 4 676 to 7 232 labels)
    (120000, 27000, 64, 5, "f32", "all"),         # more windows than chains: earlier sums
    (9001, 4099, 9, 7, "bf16", "all"),            # a last pass of three, a last window of some labels
    (15003, 2048, 5, 6, "f32", "all"),            # one block
    (4700, 3343, 10, 9, "f32", "all"),            # just above the other form's longest window
    (14465, 9643, 20, 4, "bf16", "all"),          # too few workgroups: two
    (7003, 9000, 20, 301, "f32", "one block"),    # the same; three passes over the batch, some 30000 entries beside the lists
    (300001, 14100, 30, 3, "f32", "all"),         # two rounds either way: four
    (150001, 30000, 60, 5, "bf16", "all"),
    (230001, 20640, 40, 4, "f32", "all"),         # the longest windows
    (300001, 14100, 30, 2, "bf16", "one block"),  # ... a block with all connections, beyond LDS
]


@pytest.mark.parametrize("m,d,k,b,storage,reach", CASES)
def test_places_of_the_weight_gradient(orc, m, d, k, b, storage, reach, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_BOTH", "on")
    monkeypatch.setenv("USL_TUNE_BWI_ROWS", "128")
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=760 + CASES.index((m, d, k, b, storage, reach)))
    print("backward", m, d, k, b, storage, reach, flush=True)
    idx, W, x, g = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg), wl.gen_g(cfg)
    if reach == "one block":
        idx[:] = (idx[:, :1] % 1024 + np.arange(k, dtype=np.int32) * (1024 // k)) % 1024   # distinct within a row
    L = usl.Layer(m, d, k, b, storage)
    run_and_compare(orc, L, gu, cfg, idx, W, x, g, b, max(1, b // 2))
    L.close()
