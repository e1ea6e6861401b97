"""A path long enough that its levels, one workgroup's each, take longer than a
workgroup without work waits for a record (10 s), then levels that need every
workgroup."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


def test_wide_levels_after_a_long_path(ctx):
    path, wide = 8_000_000, 200_000
    rng = np.random.default_rng(2)
    n = path + 1 + wide
    fan = np.stack([np.full(5000, path), path + 1 + np.arange(5000)], 1)
    rest = path + 1 + np.stack([rng.integers(0, 5000, 400_000), rng.integers(0, wide, 400_000)], 1)
    g = gg.gen_edges(n, np.concatenate([np.stack([np.arange(path), np.arange(1, path + 1)], 1),
                                        fan, rest]))
    want = oracle.sssp(g, 0)
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    try:
        got, st = D.dawn_sssp(ctx, h, 0)
        assert np.array_equal(got, want)
        assert st["levels"] == want.max() + 1
    finally:
        D.dawn_graph_release(ctx, h)
