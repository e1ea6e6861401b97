"""The autotuner leaves knobs alone that the chosen driver, or a batch run in one
launch, does not read."""
import pytest

import graphgen as gg
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu

LEVEL = ("block", "big_degree", "medium_edges", "medium_groups")
STEP = ("batch_alpha", "batch_big_degree", "batch_sparse_words")


@pytest.mark.parametrize("name", ["rmat12", "grid128"])
@pytest.mark.parametrize("k", [40, 600])
def test_knobs_without_effect_stay(ctx, name, k):
    g, _ = gg.load_config(name)
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    odd = dict(block=512, big_degree=777, graph_levels=6, medium_edges=5000, medium_groups=5,
               batch_alpha=3.0, batch_big_degree=99, batch_sparse_words=3)
    try:
        before = D.dawn_set_params(ctx, h, driver=3, **odd)
        best = D.dawn_autotune(ctx, h, gg.sample_sources(g.meta["wcc_nodes"], k, 7), what=3)
        if best["driver"] == 3:
            for knob in LEVEL + ("graph_levels",):
                assert best[knob] == before[knob], knob
        if k <= 512:
            for knob in STEP:
                assert best[knob] == before[knob], knob
    finally:
        D.dawn_graph_release(ctx, h)
