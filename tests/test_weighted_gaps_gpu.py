"""Weighted runs with stretches of distances far apart: however many buckets a
run needs, it ends and its rows equal the oracle's.  Long heavy paths tied to,
beside, or reached through a dense light part, and heavy-tailed weights."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


def _run(ctx, g, w, sources):
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    try:
        D.dawn_graph_set_weights(ctx, h, w)
        for s in sources:
            want = oracle.wsssp(g, w, int(s))
            got, st = D.dawn_sssp_weighted(ctx, h, int(s))
            assert np.array_equal(got.astype(np.int64), want)
            assert st["reached"] == (want >= 0).sum()
    finally:
        D.dawn_graph_release(ctx, h)


def _weights(g, path, weight):
    """`weight` on the edges between nodes of the path 0 .. path, 1 elsewhere."""
    row = np.repeat(np.arange(g.n), g.out_degree())
    return np.where((row <= path) & (g.col <= path), weight, 1).astype(np.int32)


@pytest.mark.parametrize("path,weight,clique", [
    (2000, 100, 200), (1500, 10000, 250), (1500, 100000, 250), (3000, 1000, 300), (40, 1 << 22, 60)])
def test_path_and_clique(ctx, path, weight, clique):
    """A path of `path` edges whose last node belongs to a clique of light edges."""
    a, b = np.nonzero(np.triu(np.ones((clique, clique), bool), 1))
    pairs = np.concatenate([np.stack([np.arange(path), np.arange(1, path + 1)], 1),
                            path + np.stack([a, b], 1)])
    g = gg.gen_edges(path + clique, pairs, symmetrize=True)
    w = _weights(g, path, weight)
    _run(ctx, g, w, [0, path // 2, path, g.n - 1])


@pytest.mark.parametrize("joined", [False, True])
def test_path_beside_dense_part(ctx, joined):
    """The dense light part is not reached, or is reached from the path's end."""
    path, dense = 1500, 1500
    rng = np.random.default_rng(7)
    pairs = [np.stack([np.arange(path), np.arange(1, path + 1)], 1),
             path + 1 + rng.integers(0, dense, (300000, 2))]
    if joined:
        pairs.append(np.array([[path, path + 1]]))
    g = gg.gen_edges(path + 1 + dense, np.concatenate(pairs))
    _run(ctx, g, _weights(g, path, 1024), [0, path - 1])


@pytest.mark.parametrize("name", ["rmat", "uniform", "grid"])
@pytest.mark.parametrize("top", [1 << 8, 1 << 17])
def test_heavy_tails(ctx, name, top):
    """Weights spread over the logarithm of 1 .. top, most of them small."""
    g = {"rmat": lambda: gg.gen_rmat(12, 16, 4), "uniform": lambda: gg.gen_uniform(4001, 40000, 3),
         "grid": lambda: gg.gen_grid(61, 6)}[name]()
    rng = np.random.default_rng(top)
    w = np.exp(rng.random(g.m) ** 3 * np.log(top)).astype(np.int32)
    _run(ctx, g, w, [0, 4, int(np.argmax(g.out_degree())), g.n - 1])


@pytest.mark.parametrize("first", [101, 117, 133])
def test_gap_ends_anywhere_in_a_bucket(ctx, first):
    """The next distance lies at the start, in the middle or at the end of the bucket that
    is skipped to: steps of 16 consecutive lengths, with buckets some 12 wide."""
    path, clique = 24, 60
    a, b = np.nonzero(np.triu(np.ones((clique, clique), bool), 1))
    pairs = np.concatenate([np.stack([np.arange(path), np.arange(1, path + 1)], 1),
                            path + np.stack([a, b], 1)])
    g = gg.gen_edges(path + clique, pairs, symmetrize=True)
    light = np.random.default_rng(first).integers(1, 61, g.m)
    for weight in range(first, first + 16):
        heavy = _weights(g, path, weight)
        _run(ctx, g, np.where(heavy > 1, heavy, light).astype(np.int32), [0, path // 2, g.n - 1])
