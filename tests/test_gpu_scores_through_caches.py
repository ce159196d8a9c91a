"""Scores of labels with 24 slots that go through the caches (scores_through_caches in csrc/k_products.hip): rows of scores that do not begin with a
line because of m or of the array, every workgroup shape, blocks of fewer labels, a padded fan-in.  Against the oracle, and nothing beside the scores."""
import pytest
import torch

import workloads as wl
from helpers import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("env", [{}, {"USL_TUNE_SHAPE": "0"}, {"USL_TUNE_SHAPE": "1"}, {"USL_TUNE_SHAPE": "2"}, {"USL_TUNE_SHAPE": "3", "USL_TUNE_LABELS": "800"}])
@pytest.mark.parametrize("m,d,k,b,storage,shift", [(80001, 64, 24, 210, "f32", 0), (80032, 319, 20, 213, "f32", 3), (90017, 639, 23, 187, "bf16", 1)])
def test_scores(orc, m, d, k, b, storage, shift, env, monkeypatch):
    import gpu_util as gu
    from paper_2306_03725_amd import usl
    print("scores through the caches", m, d, k, b, storage, shift, env, flush=True)
    for name, v in env.items():
        monkeypatch.setenv(name, v)
    cfg = wl.custom(m, d, k, b, storage=storage, positives=1, index=1010)
    idx, W, x = wl.gen_idx(cfg), wl.gen_W(cfg), wl.gen_x(cfg)
    L = usl.Layer(m, d, k, b, storage)
    room = gu.empty((b * m + 8,)).fill_(7.0)
    out = room[shift:shift + b * m].view(b, m)
    L.forward(gu.dev(x), gu.dev(idx), gu.dev(W), out, b)
    assert_close(gu.host(out), orc.forward(x, idx, W), 1e-5, "scores")
    assert bool((room[:shift] == 7.0).all()) and bool((room[shift + b * m:] == 7.0).all())
    L.close()
