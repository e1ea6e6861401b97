"""Weights replaced while other threads' weighted runs read them: each run's row is
that of one of the two sets."""
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


def test_replaced_under_running_calls(ctx):
    g = gg.gen_rmat(15, 16, 4)
    ws = [gg.gen_weights(g, 1, 100, seed=s, symmetric=True) for s in (1, 2)]
    src = int(np.argmax(g.out_degree()))
    want = [oracle.wsssp(g, w, src) for w in ws]
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    bad, stop = [], []
    try:
        D.dawn_graph_set_weights(ctx, h, ws[0])

        def run():
            while not stop:
                got, _ = D.dawn_sssp_weighted(ctx, h, src)
                if not any(np.array_equal(got.astype(np.int64), x) for x in want):
                    bad.append(1)
        th = [threading.Thread(target=run) for _ in range(3)]
        for t in th:
            t.start()
        for i in range(30):
            D.dawn_graph_set_weights(ctx, h, ws[(i + 1) % 2])
        stop.append(1)
        for t in th:
            t.join()
        assert not bad
    finally:
        stop.append(1)
        D.dawn_graph_release(ctx, h)
