"""Served batches of at most 1024 lanes run levels of one pass, several queued at
a time: rows and level counts equal the oracle's at every row width, with queries
that join between, with more queries than a queued level looks out for, and when
the batch grows past that width while queries run."""
import time

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


def _stars():
    """In-lists of 47..49, 511..513 and 3000 entries, reached late along a path."""
    n = 9001
    rng = np.random.default_rng(1)
    e = [np.stack([np.arange(n - 1), np.arange(1, n)], 1)[:300]]
    for v, d in [(5000, 47), (5001, 48), (5002, 49), (5003, 511), (5004, 512), (5005, 513),
                 (5006, 3000)]:
        e.append(np.stack([rng.choice(4500, d, replace=False), np.full(d, v)], 1))
    e.append(rng.integers(0, n, (20000, 2)))
    return gg.gen_edges(n, np.concatenate(e))


GRAPHS = {
    "stars": _stars,
    "rmat": lambda: gg.gen_rmat(12, 32, 5),
    "grid": lambda: gg.gen_grid(61, 7, shortcut_frac=0.0),
    # enough row words for levels queued ahead at any width
    "wide": lambda: gg.gen_grid(420, 330, shortcut_frac=0.002),
    "path": lambda: gg.gen_edges(1500, np.stack([np.arange(1499), np.arange(1, 1500)], 1)),
}


def _run(ctx, h, g, parts, pause=0.0):
    import torch
    outs, tickets = [], []
    for src in parts:
        out = torch.full((len(src), g.n), 9, dtype=torch.int32, device="cuda")
        tickets.append(D.dawn_serve_submit(ctx, h, src, out))
        outs.append(out)
        time.sleep(pause)
    stats = []
    for t in tickets:
        st, q = D.dawn_serve_wait(ctx, t, 60000)
        assert st == D.DAWN_OK
        stats.append(q)
    torch.cuda.synchronize()
    for src, out, q in zip(parts, outs, stats):
        want = oracle.mssp(g, src, threads=8)
        assert np.array_equal(out.cpu().numpy(), want), len(src)
        assert q["levels"] == want.max() + 1


@pytest.fixture(params=sorted(GRAPHS))
def graph(ctx, request):
    g = GRAPHS[request.param]()
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    yield g, h
    D.dawn_graph_release(ctx, h)


def _sources(g, k, seed):
    return np.random.default_rng(seed).integers(0, g.n, k).astype(np.int32)


@pytest.mark.parametrize("k", [1, 64, 65, 129, 257, 513, 1024, 1025])
def test_alone(ctx, graph, k):
    g, h = graph
    k = k if g.n < 100000 else min(k, 130)
    _run(ctx, h, g, [_sources(g, k, k)])


def test_joining(ctx, graph):
    g, h = graph
    _run(ctx, h, g, [_sources(g, k, i) for i, k in enumerate([3, 70, 1, 300, 2, 130, 5])], 2e-4)


def test_many_queries(ctx, graph):
    g, h = graph
    _run(ctx, h, g, [_sources(g, 2, i) for i in range(70)])


def test_grows_past_the_width(ctx, graph):
    g, h = graph
    ks = [40, 700, 900, 2000, 30, 10] if g.n < 100000 else [4, 600, 520, 6]
    for _ in range(2):
        _run(ctx, h, g, [_sources(g, k, i) for i, k in enumerate(ks)], 3e-4)
