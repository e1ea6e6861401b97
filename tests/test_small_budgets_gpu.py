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


def test_second_copy_of_weighted_rows_makes_way(dawn_lib):
    """What a budget held without the second copy of a weighted graph's rows it holds
    with it: an allocation that does not fit takes the copy back."""
    ctx = D.dawn_create(0, 64 << 20)
    try:
        g = gg.gen_rmat(13, 16, 4)
        w = gg.gen_weights(g, 1, 100, seed=3, symmetric=True)
        src = int(np.argmax(g.out_degree()))
        want = oracle.wsssp(g, w, src)
        h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
        plain = D.dawn_graph_get_info(ctx, h)["device_bytes"]
        D.dawn_graph_set_weights(ctx, h, w)
        copy = D.dawn_graph_get_info(ctx, h)["device_bytes"] - plain - 4 * g.m
        assert copy > 8 * g.m                             # the budget is plenty for it
        got, _ = D.dawn_sssp_weighted(ctx, h, src)
        assert np.array_equal(got.astype(np.int64), want)
        used, budget = D.dawn_memory(ctx)
        n = 2000                                          # a graph that fits without the copy
        m = (budget - used + copy // 2) // 8
        rng = np.random.default_rng(1)
        rp = np.linspace(0, m, n + 1).astype(np.int32)
        h2 = D.dawn_graph_upload(ctx, rp, rng.integers(0, n, int(rp[-1])).astype(np.int32))
        assert D.dawn_graph_get_info(ctx, h)["device_bytes"] == plain + 4 * g.m
        for _ in range(2):
            got, st = D.dawn_sssp_weighted(ctx, h, src)
            assert np.array_equal(got.astype(np.int64), want)
            assert st["reached"] == (want >= 0).sum()
        D.dawn_graph_release(ctx, h2)
        D.dawn_graph_set_weights(ctx, h, w)               # and it is made again
        assert D.dawn_graph_get_info(ctx, h)["device_bytes"] == plain + 4 * g.m + copy
        got, _ = D.dawn_sssp_weighted(ctx, h, src)
        assert np.array_equal(got.astype(np.int64), want)
    finally:
        D.dawn_destroy(ctx)


def test_dense_weighted_graph_with_one_queue(dawn_lib):
    """A dense graph's weighted run where the session's four sub-queues do not fit:
    it runs with one, in the memory that a launch per round took."""
    n, m = 2000, 1_000_000
    rng = np.random.default_rng(4)
    rp = np.linspace(0, m, n + 1).astype(np.int32)
    g = gg.Graph(n, rp, rng.integers(0, n, m).astype(np.int32))
    w = rng.integers(1, 101, m).astype(np.int32)
    ctx = D.dawn_create(0, 0)
    try:
        D.dawn_graph_upload(ctx, g.row_ptr, g.col)
        used = D.dawn_memory(ctx)[0]
    finally:
        D.dawn_destroy(ctx)
    ctx = D.dawn_create(0, used + 4 * m + 128 * n + 5 * m // 16)
    try:
        h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
        D.dawn_graph_set_weights(ctx, h, w)
        for s in (0, 77, n - 1):
            got, st = D.dawn_sssp_weighted(ctx, h, s)
            want = oracle.wsssp(g, w, s)
            assert np.array_equal(got.astype(np.int64), want)
            assert st["reached"] == (want >= 0).sum()
    finally:
        D.dawn_destroy(ctx)
