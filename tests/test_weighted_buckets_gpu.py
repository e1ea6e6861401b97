"""Weighted runs settle distances in buckets: rows equal the oracle's where a
bucket can go wrong (light and heavy edges of one row, gaps between distances
wider than a bucket, rows of several pieces, nodes with heavy edges only, all
weights zero or equal), and with too little memory for the second copy of the
rows."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


def _weights(g, kind, seed):
    rng = np.random.default_rng(seed)
    if kind == "uniform":
        return rng.integers(1, 101, g.m).astype(np.int32)
    if kind == "gaps":       # mostly 1, a few so heavy that buckets between lie empty
        return np.where(rng.random(g.m) < 0.05, 20000, 1).astype(np.int32)
    if kind == "heavy":      # light edges are rare
        return np.where(rng.random(g.m) < 0.02, 1, 900 + rng.integers(0, 100, g.m)).astype(np.int32)
    if kind == "zero":
        return np.zeros(g.m, np.int32)
    return np.full(g.m, 7, np.int32)


def _graph(name):
    if name == "uniform":
        return gg.gen_uniform(5001, 60000, 3)
    if name == "rmat":
        return gg.gen_rmat(13, 16, 4)
    if name == "hub":        # rows around the piece length, and a long one
        n = 4000
        rows = [(0, 63), (1, 64), (2, 65), (3, 128), (4, 3500)]
        rng = np.random.default_rng(5)
        e = [np.stack([np.full(k, u), rng.integers(0, n, k)], 1) for u, k in rows]
        e.append(np.stack([rng.integers(0, n, 12000), rng.integers(0, n, 12000)], 1))
        return gg.gen_edges(n, np.concatenate(e), drop_self=False, dedupe=False)
    return gg.gen_grid(67, 6)


def _check(ctx, g, w, sources):
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    try:
        D.dawn_graph_set_weights(ctx, h, w)
        for s in sources:
            want = oracle.wsssp(g, w, int(s))
            got, st = D.dawn_sssp_weighted(ctx, h, int(s))
            assert np.array_equal(got.astype(np.int64), want)
            assert st["reached"] == (want >= 0).sum()
            assert st["source_edges"] == g.out_degree()[want >= 0].sum()
    finally:
        D.dawn_graph_release(ctx, h)


@pytest.mark.parametrize("kind", ["uniform", "gaps", "heavy", "zero", "equal"])
@pytest.mark.parametrize("name", ["uniform", "rmat", "hub", "grid"])
def test_buckets(ctx, name, kind):
    g = _graph(name)
    w = _weights(g, kind, 11)
    _check(ctx, g, w, [0, 4, int(np.argmax(g.out_degree())), g.n - 1])


def test_without_room_for_the_copy(dawn_lib):
    """A budget with room for the weights but not, out of plenty, for a second
    copy of the rows: the same distances."""
    g = _graph("rmat")
    w = _weights(g, "uniform", 12)
    ctx = D.dawn_create(0, 16 << 20)
    try:
        _check(ctx, g, w, [0, int(np.argmax(g.out_degree()))])
    finally:
        D.dawn_destroy(ctx)
