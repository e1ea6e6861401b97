"""Narrow batches (at most 512 sources) run all their levels in one launch: rows
equal the oracle's at every row width, on graphs with in-lists around the
chunk and whole-wave lengths, on runs deeper than the level planes first
given, and when such runs and wider ones take turns on a workspace."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


def _stars():
    """In-lists of 47..49, 511..513 and 3000 entries, their sources reached late."""
    n = 9001
    rng = np.random.default_rng(1)
    e = [np.stack([np.arange(n - 1), np.arange(1, n)], 1)[:300]]      # a path first
    for v, d in [(5000, 47), (5001, 48), (5002, 49), (5003, 511), (5004, 512), (5005, 513),
                 (5006, 3000)]:
        e.append(np.stack([rng.choice(4500, d, replace=False), np.full(d, v)], 1))
    e.append(rng.integers(0, n, (20000, 2)))
    return gg.gen_edges(n, np.concatenate(e))


GRAPHS = {
    "stars": _stars,
    "rmat": lambda: gg.gen_rmat(13, 16, 5),
    "uniform": lambda: gg.gen_uniform(4097, 30000, 6),
    "grid": lambda: gg.gen_grid(61, 7, shortcut_frac=0.0),
    "path": lambda: gg.gen_edges(1500, np.stack([np.arange(1499), np.arange(1, 1500)], 1)),
    "one": lambda: gg.gen_edges(1, np.zeros((0, 2), np.int64)),
}


@pytest.fixture(scope="module")
def graphs(ctx):
    made = {}

    def get(name):
        if name not in made:
            g = GRAPHS[name]()
            src = np.random.default_rng(9).integers(0, g.n, 520).astype(np.int32)
            made[name] = (g, D.dawn_graph_upload(ctx, g.row_ptr, g.col), src,
                          oracle.mssp(g, src, threads=8))
        return made[name]
    yield get
    for g, h, _, _ in made.values():
        D.dawn_graph_release(ctx, h)


@pytest.mark.parametrize("k", [1, 64, 65, 128, 129, 256, 257, 512, 513])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_row_widths(ctx, graphs, name, k):
    g, h, src, want = graphs(name)
    got, st = D.dawn_mssp(ctx, h, src[:k])
    assert np.array_equal(got, want[:k])
    assert st["levels"] == want[:k].max() + 1
    assert st["reached"] == (want[:k] >= 0).sum()
    assert st["source_edges"] == ((want[:k] >= 0).astype(np.int64) @ g.out_degree()).sum()


@pytest.mark.parametrize("name", ["stars", "grid", "path"])
def test_fresh_graph_grows_planes(ctx, name):
    g = GRAPHS[name]()
    src = np.arange(0, g.n, max(1, g.n // 70)).astype(np.int32)[:70]
    want = oracle.mssp(g, src, threads=8)
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    try:
        for _ in range(2):
            got, _st = D.dawn_mssp(ctx, h, src)
            assert np.array_equal(got, want)
    finally:
        D.dawn_graph_release(ctx, h)


def test_turns_on_one_workspace(ctx, graphs):
    import torch
    g, h, src, want = graphs("rmat")
    out = torch.full((520, g.n), 9, dtype=torch.int32, device="cuda")
    dsrc = torch.from_numpy(src).cuda()
    for k in (520, 3, 520, 200, 64, 520, 1):
        D.dawn_mssp(ctx, h, src[:k], out=out[:k])
        assert np.array_equal(out[:k].cpu().numpy(), want[:k]), k
        out.fill_(9)
        status = torch.full((1,), 7, dtype=torch.int32, device="cuda")
        D.dawn_mssp_device(ctx, h, dsrc[:k], out[:k], status=status)
        assert np.array_equal(out[:k].cpu().numpy(), want[:k]), k
        assert int(status.item()) == D.DAWN_OK
        if k < 520:
            assert bool((out[k:] == 9).all())
        bad = dsrc[:k].clone()
        bad[k // 2] = g.n
        D.dawn_mssp_device(ctx, h, bad, out[:k], status=status)
        assert int(status.item()) == D.DAWN_E_INVALID_ARG
