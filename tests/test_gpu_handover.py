"""GPU parity of multi-source runs that start in a tile and go on on copies of the
graph: handed over early and late, before anything is left to do, with short and
queued rows in the frontier, vertex counts that are and are not multiples of 64,
weighted and hop counts, with and without a reverse graph."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import INF32, announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu


def _hubs(wk):
    """A ring with rows of 3 edges, and hubs of 40, 300 and 3000."""
    n = 4099
    rng = np.random.default_rng(3)
    src = np.concatenate([np.repeat(np.arange(n), 2), np.full(3000, 5), np.repeat(np.arange(9, 4000, 133), 40),
                          np.repeat([77, 2222, 3333], 300)])
    dst = np.concatenate([np.stack([(np.arange(n) + 1) % n, (np.arange(n) + 7) % n], 1).ravel(),
                          rng.integers(0, n, src.size - 2 * n)])
    w = rng.integers(1, 50, src.size)
    return graphgen.from_edges(n, src, dst, w.astype(np.uint32) if wk == "u32" else
                               (w / np.float32(7)).astype(np.float32), wk)


GRAPHS = {
    "grid": lambda wk: graphgen.grid(64, 80, 0.01, 3, weights="u32" if wk == "u32" else "f32unit"),
    "ragged grid": lambda wk: graphgen.grid(37, 41, 0.02, 4, weights="u32" if wk == "u32" else "f32unit"),
    "hubs": _hubs,
    "sparse er": lambda wk: graphgen.er(20011, 70001, 5, weights="u32" if wk == "u32" else "f32lognormal"),
    "er": lambda wk: graphgen.er(9001, 72001, 6, weights="u32" if wk == "u32" else "f32lognormal"),
    "rmat": lambda wk: graphgen.rmat(12, 4, 7, weights="u32" if wk == "u32" else "f32lognormal"),
}
TUNINGS = [dict(), dict(tile_step_launches=1), dict(tile_step_launches=2, t_lane=2, t_wave=64, t_chunk=256),
           dict(tile_step_launches=3, t_lane=30, grid=3, wg_threads=256), dict(tile_step_launches=200)]


def _run(dawn, call, csr, srcs, tg=None, **tune):
    prev = dawn.set_tuning(small_m=0, **tune)
    try:
        info = dawn.info_tensor()
        D = to_np(call(csr, srcs, info=info, tgraph=tg, check=False))
        return D, dawn.read_info(info)
    finally:
        dawn.set_tuning(**prev)


@pytest.mark.parametrize("ti", range(len(TUNINGS)))
@pytest.mark.parametrize("wk", ["u32", "f32"])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_weighted(dawn, name, wk, ti):
    g = GRAPHS[name](wk)
    csr = dawn.Csr.from_graph(g)
    k = {"er": 20, "hubs": 6}.get(name, (5, 9, 31, 32, 12)[ti])
    srcs = np.random.default_rng(ti).integers(0, g.n, k).astype(np.int32)
    srcs[0], srcs[-1] = g.n - 1, srcs[k // 2]
    announce("handover", name, wk, "k", k, TUNINGS[ti])
    for tg in (None, dawn.tgraph(csr)):
        D, i = _run(dawn, dawn.msssp, csr, srcs, tg, **TUNINGS[ti])
        assert i["converged"] == 1
        for j in range(k):
            assert_sssp_matches(g, int(srcs[j]), D[j], tag=f"{name} col {j}", check_invariants=False)


@pytest.mark.parametrize("ti", range(len(TUNINGS)))
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_hop_counts_and_counters(dawn, name, ti):
    g = GRAPHS[name]("u32")
    csr = dawn.Csr.from_graph(g)
    k = {"er": 7, "hubs": 6}.get(name, (5, 9, 31, 32, 12)[ti])
    srcs = graphgen.pick_sources(g, k, 8)
    lv = [oracle.bfs(g, int(s)) for s in srcs]
    announce("handover, hop counts", name, "k", k, TUNINGS[ti])
    for tg in (None, dawn.tgraph(csr)):
        D, i = _run(dawn, dawn.umsssp, csr, srcs, tg, **TUNINGS[ti])
        for j in range(k):
            assert np.array_equal(D[j].view(np.uint32), np.where(lv[j] < 0, INF32, lv[j]).astype(np.uint32)), j
        assert i["converged"] == 1
        assert i["steps"] == max(int(x.max()) + 1 for x in lv)
        assert i["edges_scanned"] == sum(oracle.m_reach(g, int(s)) for s in srcs)
        assert i["improvements"] == sum(int((x >= 0).sum()) - 1 for x in lv)
        assert i["frontier_entries"] == sum(int(((x >= 0) & (g.outdeg() > 0)).sum()) for x in lv)
        assert 0 < i["union_edges"] <= i["edges_scanned"] and 0 < i["union_rows"] <= i["frontier_entries"]


def test_improvements_go_on(dawn):
    """A chain of 300 steps of weight 1, and targets that every vertex of it lowers:
    each lowering in a step of its own, before and after the handover."""
    L, T, n = 300, 4, 6000
    c = np.arange(L + 1)
    src = np.concatenate([c[:-1], np.repeat(c, T), np.arange(1000, n)])
    dst = np.concatenate([c[1:], np.tile(np.arange(400, 400 + T), L + 1), np.arange(999, n - 1)])
    w = np.concatenate([np.ones(L), np.repeat(100000 - 10 * c, T), np.ones(n - 1000)]).astype(np.uint32)
    g = graphgen.from_edges(n, src, dst, w, "u32")
    csr = dawn.Csr.from_graph(g)
    for tune in (dict(), dict(tile_step_launches=1), dict(t_lane=1, t_wave=64)):
        announce("handover, improvements", tune)
        D, i = _run(dawn, dawn.msssp, csr, np.array([0, 400, 0, 401, 402], np.int32), **tune)
        assert i["improvements"] == 2 * (L + T * (L + 1)) and i["steps"] >= L + 1
        assert_sssp_matches(g, 0, D[2], tag="chain")


def test_status_without_info(dawn):
    import torch
    g = graphgen.grid(200, 210, 0.01, 9, weights="f32unit")
    csr = dawn.Csr.from_graph(g)
    srcs = graphgen.pick_sources(g, 6, 2).astype(np.int32)
    announce("handover, status")
    dawn.msssp(csr, srcs)
    assert dawn.run_status() == (0, 1)
    prev = dawn.set_tuning(barrier_ms=0)
    try:
        dawn.msssp(csr, srcs, check=False)       # gives up after the handover
        torch.cuda.synchronize()
        assert dawn.run_status() == (1, -2)
    finally:
        dawn.set_tuning(**prev)
    srcs[2] = g.n
    dawn.msssp(csr, srcs, check=False)           # ends in the tile
    torch.cuda.synchronize()
    assert dawn.run_status() == (1, -1)
    D, i = _run(dawn, dawn.msssp, csr, srcs)
    T, ti = _run(dawn, dawn.msssp, csr, srcs, mode=1)
    assert i == ti and np.array_equal(D.view(np.uint32), T.view(np.uint32))


def test_captured_calls_take_the_tile_alone(dawn):
    import torch
    g = graphgen.grid(211, 307, 0.01, 11, weights="u32")
    csr = dawn.Csr.from_graph(g)
    k = 5
    src = torch.as_tensor(graphgen.pick_sources(g, k, 1), dtype=torch.int32, device="cuda")
    out = torch.empty((k, g.n), dtype=torch.uint32, device="cuda")
    ws = dawn.workspace(dawn.msssp_workspace_bytes(g.n, g.m, k))
    info = dawn.info_tensor()
    announce("handover, captured")
    dawn.msssp(csr, src, out=out, ws=ws, info=info)
    eager = to_np(out).copy()
    cg = torch.cuda.CUDAGraph()
    with torch.cuda.graph(cg):
        dawn.msssp(csr, src, out=out, ws=ws, info=info, check=False)
    for rep in range(3):
        out.zero_()
        cg.replay()
        torch.cuda.synchronize()
        assert dawn.read_info(info)["converged"] == 1
        assert np.array_equal(to_np(out), eager)
        dawn.msssp(csr, src, ws=ws)
