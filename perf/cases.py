"""The calls this library is used for, as cases that can be timed.

Every case makes a seeded synthetic graph on the GPU, keeps what a program would
keep between calls (the resident CSR, the reverse graph, the workspace, the
output buffer, a batch or tile handle) and runs one call through the Python
binding.  The graph families and sizes are those of the benchmark and its
workload recipes: directed Erdos-Renyi graphs with 8 edges per vertex, R-MAT
graphs with 16 (scales 14 to 22), and 4-neighbour grids with 1 % of the pairs
deleted (path lengths of thousands of edges).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2306_07872_amd as dawn

INF32 = 0xFFFFFFFF
I32MAX = 0x7FFFFFFF

EXACT_WORK = 6e10         # edges x sources x rounds that exact() goes through at most


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # The smallest call: one source on a 1000-vertex graph, as a program
        # asks it thousands of times; latency is everything.
        dict(name="sssp_er1k_u32", call="sssp", family="er", n=1000, m=8000, wtype="u32"),
        # An ordinary small graph, ragged sizes, fp32 weights.
        dict(name="sssp_er15k_f32", call="sssp", family="er", n=15013, m=120104, wtype="f32"),
        # One source on a graph with signed weights (no negative cycle).
        dict(name="sssp_rmat18_i32", call="sssp", family="rmat", n=1 << 18, m=1 << 22, wtype="i32"),
        # One source on the road-like graph: thousands of steps with a thin frontier.
        dict(name="sssp_grid2048_f32", call="sssp", family="grid", n=2048 * 2048, cols=2048, wtype="f32"),
        # One source on the largest graph.
        dict(name="sssp_rmat22_u32", call="sssp", family="rmat", n=1 << 22, m=1 << 26, wtype="u32"),
        # The benchmark's headline: 256 sources at once, reverse graph resident.
        dict(name="msssp_rmat20_k256_u32", call="msssp", family="rmat", n=1 << 20, m=1 << 24, wtype="u32",
             k=256, reverse=True),
        # An odd number of sources on a mid-sized graph, nothing kept but the CSR.
        dict(name="msssp_rmat16_k37_f32", call="msssp", family="rmat", n=1 << 16, m=1 << 20, wtype="f32",
             k=37, reverse=False),
        # A few sources on a road-like graph.
        dict(name="msssp_grid1000_k8_f32", call="msssp", family="grid", n=1000 * 1021, cols=1021, wtype="f32",
             k=8, reverse=False),
        # All pairs of a small graph.
        dict(name="apsp_er1531_u32", call="apsp", family="er", n=1531, m=12248, wtype="u32"),
        # Hop counts from 256 sources, reverse graph resident.
        dict(name="hops_rmat20_k256", call="hops", family="rmat", n=1 << 20, m=1 << 24, wtype="unit",
             k=256, reverse=True),
        # 64 uneven graphs, one source each, in one launch.
        dict(name="batch_er64_f32", call="batch", family="er", count=64, nlo=10_000, nhi=1_000_000, wtype="f32"),
        # A serving session: queries share a tile that runs a few steps at a time.
        dict(name="tile_rmat18_q24_f32", call="tile", family="rmat", n=1 << 18, m=1 << 22, wtype="f32",
             k=24, reverse=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _family(rng, mlo, mhi, grid_most=1 << 24):
    """A graph's family and sizes; grids of at most grid_most edges."""
    m = _log(rng, mlo, mhi)
    family = rng.choice(["er", "rmat", "grid"])
    if family == "er":
        return dict(family=family, n=max(2, m // 8 + rng.randrange(8)), m=m)
    if family == "rmat":
        scale = max(8, min(22, round(math.log2(m / 16))))
        return dict(family=family, n=1 << scale, m=m)
    side = max(8, math.isqrt(min(m, grid_most) // 4))
    cols = side + rng.randrange(max(1, side // 4))
    return dict(family=family, n=side * cols, cols=cols)


def draw(rng):
    call = rng.choice(["sssp", "sssp", "msssp", "msssp", "apsp", "hops", "batch", "tile"])
    if call == "sssp":
        return dict(call=call, **_family(rng, 4e3, 3.2e7), wtype=rng.choice(["u32", "f32", "i32", "unit"]))
    if call == "msssp":
        c = _family(rng, 1e4, 8e6, 2_000_000)
        most = 12 if c["family"] == "grid" else 256  # grids take thousands of steps
        return dict(call=call, **c, wtype=rng.choice(["u32", "f32"]), k=_log(rng, 2, most),
                    reverse=rng.random() < 0.5)
    if call == "apsp":
        n = _log(rng, 100, 2500)
        return dict(call=call, family="er", n=n, m=8 * n + rng.randrange(7), wtype=rng.choice(["u32", "f32", "unit"]))
    if call == "hops":
        c = _family(rng, 1e5, 1.6e7, 1_000_000)
        most = 12 if c["family"] == "grid" else 256
        return dict(call=call, **c, wtype="unit", k=_log(rng, 8, most), reverse=rng.random() < 0.5)
    if call == "batch":
        hi = _log(rng, 20_000, 500_000)
        return dict(call=call, family="er", count=rng.randrange(4, 65), nlo=_log(rng, 1_000, hi // 2), nhi=hi,
                    wtype=rng.choice(["u32", "f32"]))
    scale = rng.randrange(14, 20)
    return dict(call="tile", family="rmat", n=1 << scale, m=rng.choice([8, 16, 32]) << scale,
                wtype=rng.choice(["u32", "f32"]), k=rng.randrange(2, 65), reverse=rng.random() < 0.5)


# ---------------------------------------------------------------------------
# graphs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _edges(case, n, m, gen):
    """(source, target) ids of the directed edges, int64."""
    dev = "cuda"
    if case["family"] == "er":
        src = torch.randint(0, n, (m,), generator=gen, device=dev)
        dst = (src + torch.randint(1, max(2, n), (m,), generator=gen, device=dev)) % n  # no self-loops
        return src, dst
    if case["family"] == "rmat":  # (a, b, c, d) = (0.57, 0.19, 0.19, 0.05), relabelled
        scale = n.bit_length() - 1
        src = torch.zeros(m, dtype=torch.int64, device=dev)
        dst = torch.zeros(m, dtype=torch.int64, device=dev)
        for _ in range(scale):
            p = torch.rand(m, generator=gen, device=dev)
            src = src * 2 + (p >= 0.76)
            dst = dst * 2 + (((p >= 0.57) & (p < 0.76)) | (p >= 0.95))
        keep = src != dst
        label = torch.randperm(n, generator=gen, device=dev)
        return label[src[keep]], label[dst[keep]]
    cols = case["cols"]
    v = torch.arange(n, device=dev)
    right, down = v[v % cols != cols - 1], v[: n - cols]
    a, b = torch.cat([right, down]), torch.cat([right + 1, down + cols])
    keep = torch.rand(a.numel(), generator=gen, device=dev) >= 0.01
    a, b = a[keep], b[keep]
    return torch.cat([a, b]), torch.cat([b, a])


def _weights(case, m, src, dst, n, gen):
    wt = case["wtype"]
    if wt == "unit":
        return torch.zeros(1, dtype=torch.int32, device="cuda").view(torch.uint32)
    if wt == "f32":
        if case["family"] == "grid":  # uniform on (0, 1]
            return 1.0 - torch.rand(m, generator=gen, device="cuda")
        return torch.randn(m, generator=gen, device="cuda").exp_()  # lognormal(0, 1)
    w = torch.randint(1, 256, (m,), generator=gen, device="cuda")
    if wt == "i32":  # potentials keep every cycle's weight: no negative cycle, many negative edges
        p = torch.randint(0, 101, (n,), generator=gen, device="cuda")
        return (w + p[src] - p[dst]).to(torch.int32)
    return w.to(torch.int32).view(torch.uint32)


def _graph(case, n, m, gen):
    """A CSR with rows sorted by column, and one edge's source per entry."""
    src, dst = _edges(case, n, m, gen)
    key, _ = torch.sort(src * n + dst)
    src, dst = key // n, key % n
    del key
    m = int(src.numel())
    rowptr = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(src, minlength=n), 0)
    w = _weights(case, m, src, dst, n, gen)
    csr = dawn.Csr(rowptr.to(torch.int32), dst.to(torch.int32), w, n, m, case["wtype"])
    return csr, src.to(torch.int32)


def _sources(csr, k, gen):
    """k sources, uniform among the vertices with out-edges."""
    deg = csr.rowptr[1:] - csr.rowptr[:-1]
    cand = torch.nonzero(deg > 0).flatten()
    return cand[torch.randint(0, cand.numel(), (k,), generator=gen, device="cuda")].to(torch.int32)


def _batch_sizes(case):
    u = np.random.default_rng(case["count"] + case["nhi"]).random(case["count"])
    lo, hi = math.log(case["nlo"]), math.log(case["nhi"])
    return [int(round(math.exp(lo + (hi - lo) * x))) for x in u]


def _inputs(case, seed):
    """The graphs and sources of a case: [(csr, edge sources, query sources)]."""
    gen = _gen(seed)
    if case["call"] == "batch":
        out = []
        for n in _batch_sizes(case):
            csr, src = _graph(case, n, 8 * n, gen)
            out.append((csr, src, _sources(csr, 1, gen)))
        return out
    csr, src = _graph(case, case["n"], case.get("m", 0), gen)
    k = case["n"] if case["call"] == "apsp" else case.get("k", 1)
    s = torch.arange(k, dtype=torch.int32, device="cuda") if case["call"] == "apsp" else _sources(csr, k, gen)
    return [(csr, src, s)]


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def prepare(case, seed):
    graphs = _inputs(case, seed)
    call = case["call"]
    if call == "batch":
        batch = dawn.Batch([g for g, _, _ in graphs])
        sources = torch.cat([s for _, _, s in graphs])
        out = torch.empty(batch.total_n, dtype=dawn.dist_dtype(case["wtype"]), device="cuda")
        return dict(call=call, batch=batch, sources=sources, out=out)
    csr, _, sources = graphs[0]
    st = dict(call=call, csr=csr, sources=sources)
    if case.get("reverse"):
        st["tgraph"] = dawn.tgraph(csr)
    if call == "sssp":
        st["source"] = int(sources[0])
        st["out"] = torch.empty(csr.n, dtype=dawn.dist_dtype(csr.wtype), device="cuda")
        st["ws"] = dawn.workspace(dawn.sssp_workspace_bytes(csr.n, csr.m))
    elif call in ("msssp", "hops") and case.get("reverse"):
        size = dawn.umsssp_workspace_bytes if call == "hops" else dawn.msssp_workspace_bytes
        st["out"] = torch.empty((case["k"], csr.n), dtype=dawn.dist_dtype(csr.wtype), device="cuda")
        st["ws"] = dawn.workspace(size(csr.n, csr.m, case["k"]))
    elif call == "tile":
        st["tile"] = dawn.Tile(csr, 64)
        if case.get("reverse"):
            st["tile"].set_tgraph(st["tgraph"])
        st["queries"] = [int(s) for s in sources.cpu()]
        st["out"] = torch.empty((case["k"], csr.n), dtype=dawn.dist_dtype(csr.wtype), device="cuda")
    return st


def run(st):
    out = _call(st)
    # whole distances as int32 words: torch indexes and sums those
    return out.view(torch.int32) if out.dtype == torch.uint32 else out


def _call(st):
    call = st["call"]
    if call == "sssp":
        return dawn.sssp(st["csr"], st["source"], out=st["out"], ws=st["ws"])
    if call == "msssp":
        return dawn.msssp(st["csr"], st["sources"], out=st.get("out"), ws=st.get("ws"), tgraph=st.get("tgraph"))
    if call == "hops":
        return dawn.umsssp(st["csr"], st["sources"], out=st.get("out"), ws=st.get("ws"), tgraph=st.get("tgraph"))
    if call == "apsp":
        return dawn.apsp(st["csr"])
    if call == "batch":
        return st["batch"].run(st["sources"], out=st["out"])
    # a session: admit the queries, run four steps at a time until all are done,
    # read each answer and give its column back
    tile, queries = st["tile"], st["queries"]
    for col, s in enumerate(queries):
        tile.admit(col, s)
    while True:
        done = dawn.done_columns(tile.run(4).cpu().numpy(), tile.k)
        if len(done) == len(queries):
            break
    for col in range(len(queries)):
        tile.read(col, out=st["out"][col])
        tile.evict(col)
    return st["out"]


# ---------------------------------------------------------------------------
# what a pass cannot do without, and what it should return
# ---------------------------------------------------------------------------

def _sizes(case):
    """(vertices, edges, distances) of one pass."""
    if case["call"] == "batch":
        n = case["count"] * (case["nhi"] - case["nlo"]) / math.log(case["nhi"] / case["nlo"])
        return n, 8 * n, n
    n = case["n"]
    m = case["m"] if "m" in case else 4 * n
    k = n if case["call"] == "apsp" else case.get("k", 1)
    return n, m, k * n


def work(case):
    n, m, out = _sizes(case)
    # the CSR is read once and every distance written once; an add and a
    # compare per edge and source
    per_edge = 4 if case["wtype"] == "unit" else 8
    return {"bytes": 4 * (n + 1) + per_edge * m + 4 * out, "flops": 2 * m * out / n}


def _exact_rows(csr, src, sources):
    """Distances [k, n] by Bellman-Ford rounds over all edges until nothing
    changes: fp64 sums for fp32 weights, int64 for whole ones."""
    n, k = csr.n, int(sources.numel())
    fl = csr.wtype == "f32"
    if csr.wtype == "unit":
        w = torch.ones(csr.m, dtype=torch.int64, device="cuda")
    else:
        w = csr.w.to(torch.float64) if fl else csr.w.view(torch.int32).to(torch.int64)
    big = math.inf if fl else 1 << 60
    dst = csr.colidx[: csr.m].to(torch.int64)
    src = src.to(torch.int64)
    order = torch.argsort(dst, stable=True)
    deg = torch.bincount(dst, minlength=n)
    rows = []
    if int(deg.max()) <= 8:  # grids: a table of each vertex's in-edges
        width = int(deg.max())
        first = torch.cumsum(deg, 0) - deg
        slot = torch.arange(csr.m, device="cuda") - first[dst[order]]
        tsrc = torch.zeros((n, width), dtype=torch.int64, device="cuda")
        tw = torch.full((n, width), big, dtype=w.dtype, device="cuda")
        tsrc[dst[order], slot] = src[order]
        tw[dst[order], slot] = w[order]
        for s in sources.tolist():
            d = torch.full((n,), big, dtype=w.dtype, device="cuda")
            d[s] = 0
            while True:
                for _ in range(64):
                    e = torch.minimum(d, (d[tsrc] + tw).amin(1))
                    d, last = e, d
                if torch.equal(d, last):
                    break
            rows.append(d)
        return torch.stack(rows)
    for lo in range(0, k, 16):
        part = sources[lo:lo + 16].to(torch.int64)
        b = part.numel()
        # fp64 bits of values >= 0 order like int64, whose minimum is exact
        d = torch.full((b, n), big, dtype=w.dtype, device="cuda")
        d[torch.arange(b, device="cuda"), part] = 0
        while True:
            e = d.clone()
            for j in range(b):
                cand = d[j][src] + w
                if fl:
                    e[j].view(torch.int64).scatter_reduce_(0, dst, cand.view(torch.int64), "amin")
                else:
                    e[j].scatter_reduce_(0, dst, cand, "amin")
                e[j][part[j]] = 0
            if torch.equal(d, e):
                break
            d = e
        rows.append(d)
    return torch.cat(rows)


def exact(case, seed):
    n, m, out = _sizes(case)
    rounds = 2 * (n / case["cols"] + case["cols"]) if case["family"] == "grid" else 40
    if m * (out / n) * rounds > EXACT_WORK * (6 if case["family"] == "grid" else 1):
        return None  # over about 20 seconds
    graphs = _inputs(case, seed)
    parts = []
    for csr, src, s in graphs:
        d = _exact_rows(csr, src, s)
        if case["wtype"] != "f32":  # whole numbers, unreachable ones as the library writes them
            inf = I32MAX if case["wtype"] == "i32" else INF32
            d = torch.where(d >= 1 << 59, inf, d).to(torch.int32)
        parts.append(d)
    if case["call"] == "batch":
        return torch.cat([p[0] for p in parts])
    return parts[0][0] if case["call"] == "sssp" else parts[0]
