"""What a user of this framework has it do, as timed cases.

Each case is one program's pass through the public entry points of
``paper_2208_04514_amd.dawn`` on a seeded synthetic graph: distances from a few
sources one call at a time, a batch of sources in one call, all pairs of a
component, weighted distances, and a burst of served queries.  The graph kinds
are those of ``graphgen`` (directed uniform, R-MAT, damaged grid), built here
on the GPU so that a case is ready quickly; sizes are the bench's and tests'
workloads, or of the same order with odd node counts.

``listed()`` names the cases, ``draw(rng)`` gives another of the same ranges,
``prepare``/``run`` hold and do the work, ``work`` says what a pass cannot do
without, and ``exact`` gives the distances from plain torch in 64 bits.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2208_04514_amd import dawn

DEV = "cuda"

# ------------------------------------------------------------------- cases --


def listed() -> list[dict]:
    return [
        # the smallest calls: a 4096-node graph queried one source at a time,
        # where the latency of a call is everything
        dict(name="sssp_uniform4096", op="sssp", kind="uniform", n=4096, deg=8, k=8, host=False),
        # scale-free graph of the headline size, single sources, rows kept on the device
        dict(name="sssp_rmat20", op="sssp", kind="rmat", n=1 << 20, deg=16, k=16, host=False),
        # directed graph of an odd size whose rows go to numpy (the default output)
        dict(name="sssp_uniform_host", op="sssp", kind="uniform", n=300007, deg=8, k=4, host=True),
        # road-like grid with a few shortcuts: some 130 levels of middling frontiers
        dict(name="sssp_grid2048", op="sssp", kind="grid", rows=2048, cols=2048,
             shortcut=0.001, k=2, host=False),
        # road-like grid without shortcuts, odd sides: thousands of small levels
        dict(name="sssp_grid1023_long", op="sssp", kind="grid", rows=1023, cols=1025,
             shortcut=0.0, k=1, host=False),
        # many sources in one call, the widest batch
        dict(name="mssp_rmat18_4096", op="mssp", kind="rmat", n=1 << 18, deg=16, k=4096,
             host=False),
        # a few sources in one call (one 64-lane word), odd node count, rows to numpy
        dict(name="mssp_rmat17_37", op="mssp", kind="rmat", n=100003, deg=16, k=37, host=True),
        # a batch of middling width queued on the caller's stream, on a road-like grid
        dict(name="mssp_device_grid512_200", op="mssp_device", kind="grid", rows=512, cols=512,
             shortcut=0.001, k=200, host=False),
        # all pairs of the largest component (n nodes; as many again by half lie outside it)
        dict(name="apsp_rmat14", op="apsp", kind="rmat", n=12463, deg=16, k=0, host=False),
        # weighted distances on a scale-free graph and on a road-like grid
        dict(name="weighted_rmat20", op="weighted", kind="rmat", n=1 << 20, deg=16, k=4,
             host=False),
        dict(name="weighted_grid1024", op="weighted", kind="grid", rows=1024, cols=1024,
             shortcut=0.001, k=2, host=False),
        # a burst of queries of mixed widths on two resident graphs, device rows
        dict(name="serve_mix", op="serve", kind="rmat", n=1 << 16, deg=16, rows=512, cols=512,
             shortcut=0.001, queries=24, kmax=512, k=0, host=False),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    x = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(max(x, lo), hi)


def draw(rng) -> dict:
    op = rng.choice(["sssp", "sssp", "sssp", "mssp", "mssp", "mssp_device", "apsp", "weighted",
                     "weighted", "serve"])
    if op == "serve":
        side = _log_int(rng, 128, 512)
        return dict(op=op, kind="rmat", n=_log_int(rng, 1 << 12, 1 << 16), deg=16, rows=side,
                    cols=side + rng.randrange(-5, 6), shortcut=0.001,
                    queries=rng.randrange(4, 25), kmax=_log_int(rng, 16, 512), k=0, host=False)
    if op == "apsp":
        return dict(op=op, kind="rmat", n=_log_int(rng, 1 << 10, 12463), deg=16, k=0, host=False)
    kind = rng.choice(["rmat", "rmat", "uniform", "grid"])
    host = rng.random() < 0.3
    case = dict(op=op, kind=kind)
    if kind == "grid":
        long = op == "sssp" and rng.random() < 0.4
        side = _log_int(rng, 100, 1024 if long or op == "weighted" else
                        2048 if op == "sssp" else 512)
        n = side * side
        case.update(rows=side, cols=side + rng.randrange(-9, 10),
                    shortcut=0.0 if long else 0.001)
    else:
        n = _log_int(rng, 1 << 12, 1 << (20 if op in ("sssp", "weighted") else 18))
        case.update(n=n, deg=rng.choice([8, 16]))
    if op in ("sssp", "weighted"):
        case.update(k=rng.randrange(1, 3) if kind == "grid" else rng.randrange(1, 9),
                    host=host)
    else:
        # row counts over the whole range, the rows at most as many as the widest batch's
        kmax = min(4096, (1 << 27) // n if host or kind == "grid" else 4096)
        case.update(k=_log_int(rng, 1, max(kmax, 1)), host=host and op == "mssp")
    return case


# ------------------------------------------------------------------ inputs --


def _csr(n: int, src, dst, symmetric: bool):
    """(row_ptr, col) as int64 CUDA tensors: no loops, no repeats, rows sorted."""
    if symmetric:
        src, dst = torch.cat([src, dst]), torch.cat([dst, src])
    keep = src != dst
    key = torch.unique(src[keep] * n + dst[keep])
    s, d = key // n, key % n
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(torch.bincount(s, minlength=n), 0)
    return rp, d


def _uniform(n: int, deg: int, gen):
    m = deg * n
    src = torch.randint(0, n, (m,), generator=gen, device=DEV)
    dst = torch.randint(0, n, (m,), generator=gen, device=DEV)
    return _csr(n, src, dst, False)


def _rmat(n: int, deg: int, gen):
    """R-MAT of the next power of two, ids permuted, the nodes below n kept."""
    scale = max(1, (n - 1).bit_length())
    draws = deg << scale
    src = torch.zeros(draws, dtype=torch.int64, device=DEV)
    dst = torch.zeros(draws, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        r = torch.rand(draws, generator=gen, device=DEV)
        src = src * 2 + (r >= 0.76)
        dst = dst * 2 + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    perm = torch.randperm(1 << scale, generator=gen, device=DEV)
    src, dst = perm[src], perm[dst]
    keep = (src < n) & (dst < n)
    return _csr(n, src[keep], dst[keep], True)


def _component(n: int, deg: int, gen):
    """A symmetric R-MAT component of n nodes, and n // 3 isolated nodes, ids permuted."""
    scale = max(1, (n - 1).bit_length())
    rp, col = _rmat(1 << scale, deg, gen)
    order = torch.argsort(rp[1:] - rp[:-1], descending=True, stable=True)
    rank = torch.empty_like(order)
    rank[order] = torch.arange(order.numel(), device=DEV)      # by degree: 0 is the hub
    src = rank[torch.repeat_interleave(torch.arange(order.numel(), device=DEV),
                                       rp[1:] - rp[:-1])]
    dst = rank[col]
    keep = (src < n) & (dst < n)
    rp, col = _csr(n, src[keep], dst[keep], True)
    # what the hub does not reach is tied to it
    loose = torch.nonzero(_hops(rp, col, torch.zeros(1, dtype=torch.int64))[0] < 0).view(-1)
    src = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    perm = torch.randperm(n + n // 3, generator=gen, device=DEV)
    return _csr(n + n // 3, perm[torch.cat([src, loose])],
                perm[torch.cat([col, torch.zeros_like(loose)])], True)


def _grid(rows: int, cols: int, shortcut: float, gen):
    """4-neighbour grid with 5 % of its edges removed and uniform shortcuts added."""
    ids = torch.arange(rows * cols, device=DEV).view(rows, cols)
    src = torch.cat([ids[:, :-1].reshape(-1), ids[:-1].reshape(-1)])
    dst = torch.cat([ids[:, 1:].reshape(-1), ids[1:].reshape(-1)])
    e = src.numel()
    keep = torch.randperm(e, generator=gen, device=DEV)[int(0.05 * e):]
    src, dst = src[keep], dst[keep]
    extra = int(shortcut * e)
    if extra:
        n = rows * cols
        src = torch.cat([src, torch.randint(0, n, (extra,), generator=gen, device=DEV)])
        dst = torch.cat([dst, torch.randint(0, n, (extra,), generator=gen, device=DEV)])
    return _csr(rows * cols, src, dst, True)


def _weights(rp, col, seed: int):
    """1 .. 100 per undirected edge: both directions get a hash of the pair."""
    n = rp.numel() - 1
    src = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    a, b = torch.minimum(src, col), torch.maximum(src, col)
    x = (a * n + b + (seed % 100003) * 7919) * 0x2545F4914F6CDD1D
    x = (x ^ ((x >> 29) & 0x7FFFFFFFF)) * 0x5851F42D4C957F2D
    return 1 + ((x >> 33) & 0x7FFFFFFF) % 100


def _pick(rp, k: int, gen):
    """k sources among the nodes that have an out-edge."""
    pool = torch.nonzero(rp[1:] > rp[:-1]).view(-1)
    return pool[torch.randint(0, pool.numel(), (k,), generator=gen, device=DEV)]


def _generator(seed: int):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed % (1 << 62))
    return gen


def _graphs(case: dict, seed: int):
    """The case's graphs, as a list of (row_ptr, col), and the generator behind them."""
    gen = _generator(seed)
    if case["op"] == "serve":
        return [_rmat(case["n"], case["deg"], gen),
                _grid(case["rows"], case["cols"], case["shortcut"], gen)], gen
    if case["kind"] == "grid":
        return [_grid(case["rows"], case["cols"], case["shortcut"], gen)], gen
    if case["op"] == "apsp":
        return [_component(case["n"], case["deg"], gen)], gen
    make = _rmat if case["kind"] == "rmat" else _uniform
    return [make(case["n"], case["deg"], gen)], gen


def _queries(case: dict, graphs, gen):
    """Served queries: (graph index, sources), widths spread over the logarithm of 1 .. kmax."""
    out = []
    for i in range(case["queries"]):
        x = (i * 0.6180339887 + 0.5) % 1.0
        k = max(1, min(case["kmax"], int(math.exp(x * math.log(case["kmax"] + 1)))))
        gi = i % 2
        out.append((gi, _pick(graphs[gi][0], k, gen)))
    return out


class _State:
    """A context with the case's graphs resident, its sources and its output rows."""

    def __init__(self, case: dict):
        self.case = case
        self.ctx = dawn.dawn_create(0)
        self.graph = []

    def upload(self, rp, col):
        h = dawn.dawn_graph_upload(self.ctx, rp.to(torch.int32).cpu().numpy(),
                                   col.to(torch.int32).cpu().numpy())
        self.graph.append(h)
        return h

    def __del__(self):
        try:
            dawn.dawn_destroy(self.ctx)
        except Exception:
            pass


def _rows(k: int, n: int, host: bool):
    if host:
        return np.full((k, n), -2, np.int32)
    return torch.full((k, n), -2, dtype=torch.int32, device=DEV)


def prepare(case: dict, seed: int) -> _State:
    st = _State(case)
    graphs, gen = _graphs(case, seed)
    op = case["op"]
    for rp, col in graphs:
        st.upload(rp, col)
    n = graphs[0][0].numel() - 1
    if op == "serve":
        st.queries = []
        for gi, src in _queries(case, graphs, gen):
            nn = graphs[gi][0].numel() - 1
            st.queries.append((st.graph[gi], src.cpu().numpy().astype(np.int32),
                               _rows(src.numel(), nn, False)))
    elif op == "apsp":
        nodes, _, _ = dawn.dawn_apsp_wcc(st.ctx, st.graph[0], query_only=True)
        st.out = _rows(nodes.size, nodes.size, False)
    else:
        src = _pick(graphs[0][0], case["k"], gen)
        if op == "weighted":
            w = _weights(*graphs[0], seed).to(torch.int32).cpu().numpy()
            dawn.dawn_graph_set_weights(st.ctx, st.graph[0], w)
        st.src = src.to(torch.int32) if op == "mssp_device" else \
            src.cpu().numpy().astype(np.int32)
        st.out = _rows(case["k"], n, case["host"])
    torch.cuda.synchronize()
    return st


def run(st: _State):
    op, ctx = st.case["op"], st.ctx
    if op == "serve":
        tickets = [dawn.dawn_serve_submit(ctx, g, src, out) for g, src, out in st.queries]
        for t in tickets:
            dawn.dawn_serve_wait(ctx, t)
        return [out for _, _, out in st.queries]
    g = st.graph[0]
    if op == "sssp":
        for i, s in enumerate(st.src):
            dawn.dawn_sssp(ctx, g, int(s), out=st.out[i])
        return st.out
    if op == "weighted":
        for i, s in enumerate(st.src):
            dawn.dawn_sssp_weighted(ctx, g, int(s), out=st.out[i])
        return st.out
    if op == "mssp":
        dawn.dawn_mssp(ctx, g, st.src, out=st.out)
        return st.out
    if op == "mssp_device":
        return dawn.dawn_mssp_device(ctx, g, st.src, st.out)
    nodes, out, _ = dawn.dawn_apsp_wcc(ctx, g, out=st.out)
    return nodes, out


# -------------------------------------------------------------------- work --


def _edges(kind: str, case: dict) -> float:
    """CSR entries, about (repeats among R-MAT draws fall with size)."""
    if kind == "grid":
        return 2 * (0.95 + case["shortcut"]) * 2 * case["rows"] * case["cols"]
    n, deg = case["n"], case["deg"]
    if kind == "uniform":
        return float(n * deg)
    full = 1 << max(1, (n - 1).bit_length())
    return 1.8 * deg * full * (n / full) ** 2


def work(case: dict) -> dict:
    op = case["op"]

    def graph_bytes(kind):
        n = case["rows"] * case["cols"] if kind == "grid" else case["n"]
        return n, 4.0 * (n + 1 + _edges(kind, case))

    n, g = graph_bytes(case["kind"])
    if op == "sssp":            # each call reads the graph and writes one row
        b = case["k"] * (g + 4.0 * n)
    elif op == "weighted":      # ... and the weights
        b = case["k"] * (g + 4.0 * _edges(case["kind"], case) + 4.0 * n)
    elif op == "apsp":          # one row per node of the component
        b = g + 4.0 * n * n
    elif op == "serve":         # both graphs once, and every query's rows
        n2, g2 = graph_bytes("grid")
        mean_k = case["kmax"] / math.log(case["kmax"] + 1)
        b = g + g2 + 4.0 * mean_k * case["queries"] * 0.5 * (n + n2)
    else:
        b = g + 4.0 * case["k"] * n
    return {"bytes": b, "flops": 0.0}


# ------------------------------------------------------------------- exact --


def _hops(rp, col, sources):
    """Level loop over the whole edge list, one source at a time."""
    n = rp.numel() - 1
    src = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    rows = []
    for s in sources.tolist():
        dist = torch.full((n,), -1, dtype=torch.int64, device=DEV)
        dist[s] = 0
        level = 0
        while True:
            cand = col[dist[src] == level]
            cand = cand[dist[cand] < 0]
            if cand.numel() == 0:
                break
            level += 1
            dist[cand] = level
        rows.append(dist)
    return torch.stack(rows)


def _weighted(rp, col, w, sources):
    """Rounds of dist[v] = min(dist[v], dist[u] + w) over every edge to the fixed point."""
    n = rp.numel() - 1
    src = torch.repeat_interleave(torch.arange(n, device=DEV), rp[1:] - rp[:-1])
    far = 1 << 60
    rows = []
    for s in sources.tolist():
        dist = torch.full((n,), far, dtype=torch.int64, device=DEV)
        dist[s] = 0
        while True:
            new = dist.scatter_reduce(0, col, dist[src] + w, "amin")
            if torch.equal(new, dist):
                break
            dist = new
        rows.append(torch.where(dist >= far, -1, dist))
    return torch.stack(rows)


def exact(case: dict, seed: int):
    op = case["op"]
    if op in ("apsp", "serve"):
        return None
    # the long grids take a pass over the edges per level
    levels = 8 if case["kind"] != "grid" else \
        60 if case["shortcut"] else case["rows"] + case["cols"]
    if case["k"] * levels * (1.0 + _edges(case["kind"], case) / 2e7) > 2e4:
        return None
    graphs, gen = _graphs(case, seed)
    rp, col = graphs[0]
    sources = _pick(rp, case["k"], gen)
    rows = _weighted(rp, col, _weights(rp, col, seed), sources) if op == "weighted" else \
        _hops(rp, col, sources)
    return rows.cpu().numpy() if case["host"] else rows
