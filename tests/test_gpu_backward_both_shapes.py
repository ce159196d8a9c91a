"""The one-pass form of usl_backward where its cut of the layer can go wrong: layers narrower than a block of features
(a window of several runs of labels), equal blocks that end off the grid of 2048 features, windows that no fan-in or
width divides, four or two instances at a time, the batch in several parts.  Against the oracle, element by element."""
import pytest

import workloads as wl
from test_gpu_backward_both import run_and_compare

pytestmark = pytest.mark.gpu

# (m, d, k, b, storage, parts of the batch)
SHAPES = [
    (900, 3, 3, 5, "f32", 1),           # 682 runs of 4 labels
    (20011, 1, 1, 9, "f32", 1),         # one feature: as many runs of 4 labels as LDS holds
    (1024, 64, 8, 16, "bf16", 3),       # 32 runs, parts of 8, 8 and no instances
    (3000, 700, 5, 9, "f32", 2),        # two runs of a ragged number of features
    (5001, 1024, 32, 6, "f32", 1),      # two runs that fill the block
    (5001, 1025, 32, 6, "bf16", 2),     # one run, just over half a block
    (4999, 2049, 17, 7, "f32", 1),      # two blocks, 1056 and 993 features
    (20011, 2500, 64, 33, "bf16", 5),   # many windows
    (9001, 10007, 48, 18, "f32", 4),    # five blocks; 4 instances at a time
    (30001, 13591, 32, 10, "f32", 2),   # the widest layer for four at a time with this fan-in ...
    (30001, 13592, 32, 11, "bf16", 2),  # ... and the narrowest for two
    (60001, 20011, 33, 5, "bf16", 1),   # rows of x and g that start anywhere
    (3, 65536, 64, 3, "f32", 1),        # fewer labels than a wavefront has lanes
]


@pytest.mark.parametrize("m,d,k,b,storage,parts", SHAPES)
def test_one_pass_backward_shapes(orc, m, d, k, b, storage, parts, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    monkeypatch.setenv("USL_TUNE_BOTH", "on")
    monkeypatch.setenv("USL_TUNE_BOTH_PARTS", str(parts))
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=700 + SHAPES.index((m, d, k, b, storage, parts)))
    print("backward", m, d, k, b, storage, parts, flush=True)
    idx, W, x, g = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg), wl.gen_g(cfg)
    L = usl.Layer(m, d, k, b, storage)
    run_and_compare(orc, L, gu, cfg, idx, W, x, g, b, max(1, b // 2))
    L.close()


# layers of many short windows, as the layer is cut by itself: sizes at which rounding the window to a multiple of four
# labels leaves fewer windows than were aimed at
MANY_WINDOWS = [(76296, 1133, 64, 5, "f32"), (300000, 1100, 32, 6, "bf16"), (500000, 1500, 64, 2, "f32"), (670000, 2048, 32, 3, "f32")]


@pytest.mark.parametrize("m,d,k,b,storage", MANY_WINDOWS)
def test_one_pass_backward_of_many_windows(orc, m, d, k, b, storage):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    cfg = wl.custom(m, d, k, b, storage=storage, positives=3, index=720)
    print("backward", m, d, k, b, storage, flush=True)
    idx, W, x, g = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg), wl.gen_g(cfg)
    L = usl.Layer(m, d, k, b, storage)
    run_and_compare(orc, L, gu, cfg, idx, W, x, g, b, max(1, b // 2))
    L.close()


@pytest.mark.parametrize("m,d,k,b,storage,parts", SHAPES)
def test_one_pass_backward_shapes_in_bank_order(orc, m, d, k, b, storage, parts, monkeypatch):
    """Layers this small keep their lists in stored order by themselves; the bank-aware order has to be right for them too."""
    monkeypatch.setenv("USL_TUNE_ROUNDS", "3")
    test_one_pass_backward_shapes(orc, m, d, k, b, storage, parts, monkeypatch)
