"""The launch-per-step kernels, where the default settings do not take them: narrow
rows in batches beside other batches, and the level kernel with its own knobs under
drivers 2 and 4.  Rows equal the oracle's."""
import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


@pytest.fixture
def kept(ctx, upload):
    """kept(name) -> (handle, graph, sources), the graph's knobs put back afterwards."""
    saved = []

    def get(name):
        h, g, src = upload(name)
        saved.append((h, D.dawn_get_params(ctx, h)))
        return h, g, src
    yield get
    for h, p in saved:
        D.dawn_set_params(ctx, h, **p)


@pytest.mark.parametrize("name", ["rmat12", "grid128ns", "uniform4096"])
@pytest.mark.parametrize("lanes", [64, 128, 256, 512])
def test_narrow_batches_side_by_side(ctx, kept, name, lanes):
    """Rows of 1, 2, 4 and 8 words, in every direction; the last batch is narrower."""
    h, g, _ = kept(name)
    srcs = gg.sample_sources(g.n, 2 * lanes + 17, 5 + lanes)
    want = oracle.mssp(g, srcs, threads=16)
    for direction in (1, 2, 3):
        D.dawn_set_params(ctx, h, batch_lanes=lanes, direction=direction)
        got, st = D.dawn_mssp(ctx, h, srcs)
        assert np.array_equal(got, want), direction
        assert st["reached"] == (want >= 0).sum()
        if direction == 1:
            assert st["pull_levels"] == 0
        if direction == 2:
            assert st["push_levels"] == 0


@pytest.mark.parametrize("name", ["rmat12", "grid128"])
@pytest.mark.parametrize("lanes", [64, 256])
def test_narrow_batch_knobs(ctx, kept, name, lanes):
    h, g, _ = kept(name)
    srcs = gg.sample_sources(g.n, 2 * lanes, 78)
    want = oracle.mssp(g, srcs, threads=16)
    base = D.dawn_set_params(ctx, h, batch_lanes=lanes)
    for knob, vals in (("batch_alpha", (1e-4, 1, 16, 1e6)), ("batch_big_degree", (64, 256, 1024)),
                       ("batch_wide_scan", (1, 16, 96, 512)), ("batch_sparse_words", (1, 2, 4))):
        for v in vals:
            D.dawn_set_params(ctx, h, **{**base, knob: v})
            got, _ = D.dawn_mssp(ctx, h, srcs)
            assert np.array_equal(got, want), f"{knob}={v}"


@pytest.mark.parametrize("name", ["rmat12", "grid128"])
@pytest.mark.parametrize("driver", [2, 4])
def test_level_kernel_knobs(ctx, kept, name, driver):
    h, g, src = kept(name)
    want = oracle.mssp(g, src[:3])
    base = D.dawn_set_params(ctx, h, driver=driver, small_n=0)
    for kw in [dict(medium_edges=e, medium_groups=m) for e in (2000, 16384, 65536) for m in (2, 8, 64)] + \
              [dict(big_degree=b) for b in (64, 256, 8192)] + \
              [dict(small_frontier_edges=e) for e in (-1, 128, 1024)] + \
              [dict(block=b, direction=d) for b in (256, 512, 1024) for d in (1, 2, 3)]:
        D.dawn_set_params(ctx, h, **{**base, **kw})
        for r, s in enumerate(src[:3]):
            got, _ = D.dawn_sssp(ctx, h, int(s))
            assert np.array_equal(got, want[r]), f"{kw} source {s}"
