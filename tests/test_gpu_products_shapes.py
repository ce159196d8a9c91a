"""Forward and weight gradient at the edges of their kernels: the fan-ins between the unrolled ones (padded slots), the
widths at which an interleaved row of 4, 2 or 1 instances stops fitting LDS, the batches around a group of instances
(the streaming forward and its tail), and every launch shape by hand.  Against the oracle, element by element."""
import pytest

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu

# (m, d, k, b, storage)
SHAPES = [(3001, 300, k, 7, st) for k, st in [(1, "f32"), (2, "bf16"), (4, "f32"), (5, "f32"), (9, "bf16"), (17, "f32"), (24, "bf16"), (25, "f32"),
                                               (47, "bf16"), (48, "f32"), (49, "f32"), (63, "bf16"), (64, "f32")]]
SHAPES += [(5003, d, 12, b, "f32") for d, b in [(10176, 5), (10239, 4), (10240, 6), (10241, 5), (20479, 3), (20481, 3), (40703, 2), (40961, 2), (65536, 1)]]
SHAPES += [(5003, d, 16, b, "bf16") for d, b in [(20352, 5), (20480, 4), (20481, 5), (40960, 3), (40961, 3), (65535, 2), (65536, 2)]]
SHAPES += [(70001, 1000, 8, b, "f32") for b in (1, 2, 3, 4, 5, 8, 9)]


def compare(orc, gu, cfg, m, d, k, b, storage):
    from paper_2306_03725_amd import usl
    idx, W, x, g = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg), wl.gen_g(cfg)
    L = usl.Layer(m, d, k, b, storage)
    d_idx, d_W, d_x, d_g = gu.dev(idx), gu.dev(W), gu.dev(x), gu.dev(g)
    out, gW = gu.empty((b, m)).fill_(float("nan")), gu.empty((m, k)).fill_(float("nan"))
    L.forward(d_x, d_idx, d_W, out, b)
    assert_close(gu.host(out), orc.forward(x, idx, W), 1e-5, "scores")
    L.backward_weight(d_g, d_x, d_idx, gW, b)
    assert_close(gu.host(gW), orc.backward_weight(g, x, idx), 1e-5, "grad_W")
    L.close()


@pytest.mark.parametrize("m,d,k,b,storage", SHAPES)
def test_products_at_their_edges(orc, m, d, k, b, storage):
    import gpu_util as gu
    print("products", m, d, k, b, storage, flush=True)
    compare(orc, gu, wl.custom(m, d, k, b, storage=storage, positives=3, index=740 + SHAPES.index((m, d, k, b, storage))), m, d, k, b, storage)


@pytest.mark.parametrize("split", [1, 3])
@pytest.mark.parametrize("shape", [0, 1, 2])
def test_products_in_every_launch_shape(orc, shape, split, monkeypatch):
    import gpu_util as gu
    monkeypatch.setenv("USL_TUNE_SHAPE", str(shape))
    monkeypatch.setenv("USL_TUNE_SPLIT", str(split))
    for q, (m, d, k, b, storage) in enumerate([(2500, 4096, 32, 13, "f32"), (2500, 15000, 20, 13, "bf16"), (2500, 40000, 64, 5, "f32")]):
        print("products", m, d, k, b, storage, shape, split, flush=True)
        compare(orc, gu, wl.custom(m, d, k, b, storage=storage, positives=3, index=790 + q), m, d, k, b, storage)


@pytest.mark.parametrize("m,d,k,b,storage", [s for s in SHAPES if s[0] * s[2] * s[3] < 1 << 21])
def test_products_at_their_edges_in_bank_order(orc, m, d, k, b, storage, monkeypatch):
    """Layers this small keep their slots in stored order by themselves; the bank-aware order has to be right for them too."""
    monkeypatch.setenv("USL_TUNE_ROUNDS", "3")
    test_products_at_their_edges(orc, m, d, k, b, storage)


@pytest.mark.parametrize("m,d,k,b,storage,split", [(700, 9000, 5, 93, "f32", 8), (1, 2000, 8, 61, "bf16", 8), (2100, 40000, 9, 31, "f32", 16),
                                                   (600, 65536, 6, 8, "f32", 8), (4100, 65536, 8, 95, "bf16", 24)])
def test_products_with_the_parts_of_the_batch_first(orc, m, d, k, b, storage, split, monkeypatch):
    """A multiple of 8 parts, and far more activations than connections: the grid's first dimension is the part."""
    import gpu_util as gu
    monkeypatch.setenv("USL_TUNE_SPLIT", str(split))
    print("products", m, d, k, b, storage, split, flush=True)
    compare(orc, gu, wl.custom(m, d, k, b, storage=storage, positives=1, index=810 + split), m, d, k, b, storage)


# Far more labels than the other tests have.  Only the last layer has more blocks of labels than workgroups fit at once (256
# compute units), so that the blocks of its last round take the batch in parts; most others take it in parts altogether.
LAST_ROUND = [(263000, 30000, 3, 9, "f32"), (300001, 36000, 2, 35, "bf16"), (262145, 40000, 1, 4, "f32"), (600011, 20000, 3, 13, "f32"),
              (270000, 65536, 2, 5, "f32"), (530000, 10000, 5, 37, "f32")]


@pytest.mark.parametrize("m,d,k,b,storage", LAST_ROUND)
def test_scores_of_the_blocks_of_a_last_round(orc, m, d, k, b, storage):
    import gpu_util as gu
    print("products", m, d, k, b, storage, flush=True)
    compare(orc, gu, wl.custom(m, d, k, b, storage=storage, positives=1, index=830), m, d, k, b, storage)


@pytest.mark.parametrize("m,d,k,b,storage", [s for s in LAST_ROUND if s[1] < 65536])
def test_losses_of_the_blocks_of_a_last_round(orc, m, d, k, b, storage, monkeypatch):
    """The sum over all workgroups, and the target bits of parts that begin within a word of 32 instances."""
    import test_gpu_train_step as steps
    case = (m, d, k, b, storage, 0, False, False)
    monkeypatch.setattr(steps, "CASES", [case])
    steps.test_train_step(orc, *case, monkeypatch)


# (parts of the batch): groups of 4, 2, 1 instances and rows in two halves; parts that begin within a word of 32 instances, parts
# of unequal size, one of a single group; one block of labels, which is then the last half, and several
IN_PARTS = [(9001, 9000, 5, 37, "f32", 3), (9001, 15000, 9, 37, "f32", 3), (9001, 15000, 9, 64, "f32", 16), (9001, 30000, 12, 37, "f32", 4),
            (9001, 65536, 8, 35, "f32", 3), (9001, 20000, 24, 70, "bf16", 5), (9001, 30001, 33, 37, "bf16", 3), (9001, 65536, 16, 37, "bf16", 37),
            (700, 9000, 20, 10, "f32", 3), (5000, 30000, 64, 5, "f32", 2), (5000, 12000, 50, 9, "bf16", 2)]


@pytest.mark.parametrize("m,d,k,b,storage,parts", IN_PARTS)
def test_scores_of_blocks_that_take_the_batch_in_parts(orc, m, d, k, b, storage, parts, monkeypatch):
    import gpu_util as gu
    monkeypatch.setenv("USL_TUNE_TAIL", str(parts))
    print("products", m, d, k, b, storage, parts, flush=True)
    compare(orc, gu, wl.custom(m, d, k, b, storage=storage, positives=1, index=832), m, d, k, b, storage)


@pytest.mark.parametrize("m,d,k,b,storage,parts", IN_PARTS)
def test_losses_of_blocks_that_take_the_batch_in_parts(orc, m, d, k, b, storage, parts, monkeypatch):
    import test_gpu_train_step as steps
    monkeypatch.setenv("USL_TUNE_TAIL", str(parts))
    case = (m, d, k, b, storage, 0, False, False)
    monkeypatch.setattr(steps, "CASES", [case])
    steps.test_train_step(orc, *case, monkeypatch)


@pytest.mark.parametrize("split", [1, 3])
@pytest.mark.parametrize("m,d,k,b,storage", [(2500, 4096, 32, 13, "f32"), (2049, 15000, 20, 13, "bf16"), (1023, 10000, 16, 30, "f32"), (1025, 20000, 32, 7, "f32")])
def test_products_with_one_label_a_lane_in_wide_workgroups(orc, m, d, k, b, storage, split, monkeypatch):
    import gpu_util as gu
    monkeypatch.setenv("USL_TUNE_SHAPE", "3")
    monkeypatch.setenv("USL_TUNE_SPLIT", str(split))
    print("products", m, d, k, b, storage, split, flush=True)
    compare(orc, gu, wl.custom(m, d, k, b, storage=storage, positives=1, index=840 + split), m, d, k, b, storage)


@pytest.mark.parametrize("m,d,k,b,storage", [(262145, 300, 12, 1, "f32"), (262144, 40000, 13, 1, "bf16"), (140000, 1000, 30, 1, "f32"), (131073, 30000, 64, 1, "bf16"),
                                             (70001, 500, 49, 1, "f32")])
def test_scores_of_one_instance_over_many_labels(orc, m, d, k, b, storage):
    """Enough labels for four rounds in flight, 4 to 16 lanes to a label."""
    import gpu_util as gu
    print("products", m, d, k, b, storage, flush=True)
    compare(orc, gu, wl.custom(m, d, k, b, storage=storage, positives=1, index=850), m, d, k, b, storage)
