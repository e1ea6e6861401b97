"""The one-launch traversal (driver 3) at the sizes where a level changes how it
runs: one workgroup, one XCD's cluster, the grid; rows cut into pieces; pull
levels of either width; several traversals on the device at once.  Rows equal
the oracle's."""
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


def _fan(edges, children, hub=0):
    """0 -> `children` nodes, whose rows hold `edges` entries in all (the first
    child's at least `hub` of them), onto distinct nodes that all point at the last."""
    first = max(hub, edges // children)
    rest = edges - first
    cnt = np.full(children, 0, np.int64)
    cnt[0] = first
    if children > 1:
        cnt[1:] = rest // (children - 1)
        cnt[1] += rest - cnt[1:].sum()
    n = 1 + children + edges + 1
    src = [np.zeros(children, np.int64), np.repeat(np.arange(1, children + 1), cnt),
           np.arange(1 + children, n - 1)]
    dst = [np.arange(1, children + 1), 1 + children + np.arange(int(cnt.sum())),
           np.full(edges, n - 1, np.int64)]
    return gg.gen_edges(n, np.stack([np.concatenate(src), np.concatenate(dst)], 1),
                        drop_self=False, dedupe=False)


def _check(ctx, g, sources, **params):
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    try:
        D.dawn_set_params(ctx, h, driver=3, small_n=0, **params)
        for s in sources:
            want = oracle.sssp(g, int(s))
            got, st = D.dawn_sssp(ctx, h, int(s), frontier_cap=64)
            assert np.array_equal(got, want)
            assert st["levels"] == want.max() + 1
            assert st["reached"] == (want >= 0).sum()
            assert st["source_edges"] == g.out_degree()[want >= 0].sum()
            hist = np.bincount(want[want >= 0])
            assert st["frontier_sizes"] == hist[:64].tolist()
            if params.get("direction") == 1:
                assert st["edges_examined"] == st["source_edges"]
    finally:
        D.dawn_graph_release(ctx, h)


# frontier edges around the bounds of one workgroup (1024) and of a cluster
# (32768), few and many rows, with and without a row of several pieces
@pytest.mark.parametrize("edges", [1023, 1024, 1025, 2049, 32767, 32768, 32769, 300000])
@pytest.mark.parametrize("children,hub", [(1, 0), (63, 0), (64, 0), (1000, 0), (500, 500)])
def test_level_widths(ctx, edges, children, hub):
    hub = hub and edges // 2
    _check(ctx, _fan(edges, min(children, edges), hub), [0, 1], direction=1)
    _check(ctx, _fan(edges, min(children, edges), hub), [0], direction=3)


@pytest.mark.parametrize("n", [63, 64, 65, 512, 65535, 65536, 65537, 70001])
@pytest.mark.parametrize("direction", [2, 3])
def test_pull_widths(ctx, n, direction):
    g = gg.gen_uniform(n, 6 * n, seed=n)
    src = gg.sample_sources(n, 3, 5)
    _check(ctx, g, src, direction=direction)
    _check(ctx, g, src, direction=direction, small_frontier_edges=-1)


def test_concurrent_traversals(ctx):
    """Sessions that share the device: each runs with the workgroups that
    started for it."""
    g = gg.gen_uniform(150001, 1200000, seed=3)
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    src = gg.sample_sources(g.n, 12, 7)
    want = oracle.mssp(g, src, threads=8)
    bad = []

    def work(i):
        for r in range(i, src.size, 4):
            for _ in range(5):
                got, _st = D.dawn_sssp(ctx, h, int(src[r]))
                if not np.array_equal(got, want[r]):
                    bad.append(r)
    try:
        th = [threading.Thread(target=work, args=(i,)) for i in range(4)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        assert not bad
    finally:
        D.dawn_graph_release(ctx, h)
