"""Rows for host memory: equal to the oracle's around the size from which they go
through pinned pieces, for pinned destinations, served, and from several threads
of one context."""
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu

# 4 x 5003 bytes a row: 419 rows are the last below 8 MiB
WIDTHS = [1, 419, 420, 523, 524, 525, 1050]


@pytest.fixture(scope="module")
def rows(ctx):
    g = gg.gen_uniform(5003, 30000, 3)
    h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
    src = np.random.default_rng(2).integers(0, g.n, max(WIDTHS)).astype(np.int32)
    yield g, h, src, oracle.mssp(g, src, threads=8)
    D.dawn_graph_release(ctx, h)


@pytest.mark.parametrize("k", WIDTHS)
def test_widths(ctx, rows, k):
    g, h, src, want = rows
    out = np.full((k + 1, g.n), 7, np.int32)
    D.dawn_mssp(ctx, h, src[:k], out=out[:k])
    assert np.array_equal(out[:k], want[:k]) and (out[k] == 7).all()


def test_pinned_destination(ctx, rows):
    import torch
    g, h, src, want = rows
    out = torch.empty((600, g.n), dtype=torch.int32, pin_memory=True).numpy()
    D.dawn_mssp(ctx, h, src[:600], out=out)
    assert np.array_equal(out, want[:600])


def test_served(ctx, rows):
    g, h, src, want = rows
    out = np.full((700, g.n), 7, np.int32)
    st, _ = D.dawn_serve_wait(ctx, D.dawn_serve_submit(ctx, h, src[:700], out), 60000)
    assert st == D.DAWN_OK and np.array_equal(out, want[:700])


def test_threads(ctx, rows):
    g, h, src, want = rows
    bad = []

    def one(i):
        k = 430 + 60 * i
        for _ in range(4):
            out = np.full((k, g.n), 7, np.int32)
            D.dawn_mssp(ctx, h, src[i:i + k], out=out)
            if not np.array_equal(out, want[i:i + k]):
                bad.append(i)

    ts = [threading.Thread(target=one, args=(i,)) for i in range(6)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
