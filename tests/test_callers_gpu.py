"""Several threads' calls of every kind at once, on several graphs: each gets its
part of the device, a workspace goes from one call's stream to another's, and every
row equals the oracle's."""
import threading

import numpy as np
import pytest

import graphgen as gg
import oracle
from paper_2208_04514_amd import dawn as D

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("threads", [2, 4, 7])
def test_mixed_calls(ctx, threads):
    import torch
    graphs = [gg.gen_rmat(14, 16, 4), gg.gen_grid(151, 6, shortcut_frac=0.0),
              gg.gen_uniform(120001, 960000, 3)]
    made = []
    for g in graphs:
        h = D.dawn_graph_upload(ctx, g.row_ptr, g.col)
        w = gg.gen_weights(g, 1, 100, seed=9, symmetric=False)
        D.dawn_graph_set_weights(ctx, h, w)
        src = gg.sample_sources(g.n, 70, 5)
        made.append((g, h, src, oracle.mssp(g, src, threads=8), oracle.wmssp(g, w, src[:4], threads=8)))
    bad = []

    def work(t):
        out = torch.empty(max(g.n for g in graphs), dtype=torch.int32, device="cuda")
        for r in range(6):
            g, h, src, want, wwant = made[(t + r) % 3]
            i = (t + 3 * r) % 4
            got, _ = D.dawn_sssp(ctx, h, int(src[i]))
            if not np.array_equal(got, want[i]):
                bad.append(("sssp", t, r))
            D.dawn_sssp(ctx, h, int(src[i + 1]), out=out[:g.n])
            if not np.array_equal(out[:g.n].cpu().numpy(), want[i + 1]):
                bad.append(("sssp device", t, r))
            got, _ = D.dawn_sssp_weighted(ctx, h, int(src[i]))
            if not np.array_equal(got.astype(np.int64), wwant[i]):
                bad.append(("weighted", t, r))
            k = (1, 30, 70)[(t + r) % 3]
            got, _ = D.dawn_mssp(ctx, h, src[:k])
            if not np.array_equal(got, want[:k]):
                bad.append(("mssp", t, r))
    try:
        th = [threading.Thread(target=work, args=(t,)) for t in range(threads)]
        for x in th:
            x.start()
        for x in th:
            x.join()
        assert not bad
    finally:
        for _, h, _, _, _ in made:
            D.dawn_graph_release(ctx, h)
