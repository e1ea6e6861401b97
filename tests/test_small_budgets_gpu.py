"""Device memory that calls take: no more than they need where a budget is small."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


def test_planes_for_the_depth_alone(dawn_lib):
    """A narrow batch's level planes: as many as its depth has bits (at least three)."""
    n = 5000
    g = gg.gen_edges(n, np.stack([np.arange(n - 1), np.arange(1, n)], 1))
    used = {}
    for levels in (6, 8, 9, 20, 40, 70):
        ctx = D.dawn_create(0, 0)
        try:
            h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
            src = np.array([n - levels], np.int32)
            got, st = D.dawn_mssp(ctx, h, src)
            assert st["levels"] == levels
            assert np.array_equal(got, oracle.mssp(g, src))
            used[levels] = D.dawn_memory(ctx)[0]
        finally:
            D.dawn_destroy(ctx)
    for levels in used:
        # (a run looks one level past its last)
        planes = max(3, int(levels).bit_length())
        assert used[levels] - used[6] == (planes - 3) * n * 8, levels
