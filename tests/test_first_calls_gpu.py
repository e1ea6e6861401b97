"""First calls on a graph, which make a workspace: its arrays are cleared before
the traversal that uses them, however busy the null stream is meanwhile."""
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("driver", [1, 2, 3, 4, "weighted"])
def test_busy_null_stream(ctx, driver):
    """The null stream is held for some 8 ms; the traversal takes several times
    that (a path: one node a level)."""
    import torch
    n = 8000 if driver == 1 else 20000
    g = gg.gen_edges(n, np.stack([np.arange(n - 1), np.arange(1, n)], 1))
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    try:
        if driver == "weighted":
            D.dawn_graph_set_weights(ctx, h, np.full(n - 1, 7, np.int32))
        else:
            D.dawn_set_params(ctx, h, driver=driver, small_n=0)
        for _ in range(2):
            torch.cuda._sleep(20_000_000)
            if driver == "weighted":
                got, _ = D.dawn_sssp_weighted(ctx, h, 0)
                assert np.array_equal(got, 7 * np.arange(n))
            else:
                got, _ = D.dawn_sssp(ctx, h, 0)
                assert np.array_equal(got, np.arange(n))
            torch.cuda.synchronize()
    finally:
        D.dawn_graph_release(ctx, h)


def test_threads_make_workspaces(ctx):
    """Eight threads' first traversals at once, on a graph of many levels."""
    g = gg.gen_grid(301, 4)
    src = gg.sample_sources(g.n, 8, 3)
    want = oracle.mssp(g, src, threads=8)
    bad = []
    for _ in range(3):
        h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
        try:
            def work(i):
                for _ in range(3):
                    got, _st = D.dawn_sssp(ctx, h, int(src[i]))
                    if not np.array_equal(got, want[i]):
                        bad.append(i)
            th = [threading.Thread(target=work, args=(i,)) for i in range(8)]
            for t in th:
                t.start()
            for t in th:
                t.join()
        finally:
            D.dawn_graph_release(ctx, h)
    assert not bad
