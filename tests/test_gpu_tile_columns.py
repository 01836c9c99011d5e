"""GPU parity of what a tile session skips and how it cuts rows: columns that
are INF already are not filled again on admission (also when admissions were
captured into a graph), weighted rows around the 16-lane-group and wavefront
limits, and hop-count pull steps around the whole-wavefront chunk limit."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu


def _run_until_done(dawn, tile, cols):
    import torch
    for _ in range(10000):
        done = tile.run(4)
        torch.cuda.synchronize()
        if cols <= set(dawn.done_columns(to_np(done), tile.k)):
            return
    raise AssertionError("tile did not finish")


@pytest.mark.parametrize("wk", ["u32", "f32lognormal"])
def test_columns_reused_with_and_without_eviction(dawn, wk):
    g = graphgen.er(3001, 24011, 21, weights=wk)
    csr = dawn.Csr.from_graph(g)
    tile = dawn.Tile(csr, 70)
    srcs = [int(s) for s in graphgen.pick_sources(g, 8, 22)]
    for i, s in enumerate(srcs):
        announce("tile column reuse", wk, "query", i)
        for col in (3, 69):
            tile.admit(col, s)
        if i % 3 == 0:
            tile.run(2)
            tile.evict(69)                # cancelled while running, then reused
            tile.run(1)
            tile.admit(69, s)
        _run_until_done(dawn, tile, {3, 69})
        for col in (3, 69):
            assert_sssp_matches(g, s, to_np(tile.read(col)), tag=f"query {i} col {col}")
        if i % 2:
            tile.evict(3)                 # the others are admitted over the old result
    tile.close()


def test_captured_admission_leaves_no_column_unfilled(dawn):
    import torch
    g = graphgen.er(2003, 16001, 31, weights="u32")
    csr = dawn.Csr.from_graph(g)
    s0, s1 = (int(s) for s in graphgen.pick_sources(g, 2, 32))
    tile = dawn.Tile(csr, 64)
    torch.cuda.synchronize()
    cg = torch.cuda.CUDAGraph()
    with torch.cuda.graph(cg):
        tile.admit(5, s0)
    for rep in range(3):
        announce("captured admission", rep)
        tile.evict(5)
        cg.replay()
        _run_until_done(dawn, tile, {5})
        assert_sssp_matches(g, s0, to_np(tile.read(5)), tag=f"replayed {rep}")
        tile.admit(5, s1)                 # over the replayed query's distances
        _run_until_done(dawn, tile, {5})
        assert_sssp_matches(g, s1, to_np(tile.read(5)), tag=f"eager {rep}")
    tile.close()


def _degree_graph(degs, wtype):
    """A ring of n vertices; vertex i has degs[i % len(degs)] out-edges in all."""
    n, rng = 40 * len(degs), np.random.default_rng(41)
    src = np.concatenate([np.full(degs[i % len(degs)], i) for i in range(n)])
    dst = rng.integers(0, n, src.size)
    first = np.concatenate([[0], np.cumsum([degs[i % len(degs)] for i in range(n)])[:-1]])
    dst[first] = (np.arange(n) + 1) % n
    w = rng.integers(1, 100, src.size)
    w = w.astype(np.uint32) if wtype == "u32" else w.astype(np.float32) / 7
    return graphgen.from_edges(n, src, dst, w, wtype)


@pytest.mark.parametrize("wtype", ["u32", "f32"])
@pytest.mark.parametrize("k", [40, 150])
def test_weighted_rows_around_the_tier_limits(dawn, wtype, k):
    g = _degree_graph([1, 8, 9, 16, 23, 24, 25, 63, 64, 65, 127, 128, 129, 256, 257, 400], wtype)
    csr = dawn.Csr.from_graph(g)
    srcs = graphgen.pick_sources(g, k, 43)
    for tune in (dict(small_m=0), dict(small_m=0, tile_t_group=0),
                 dict(small_m=0, tile_t_group=30, tile_t_wave=32, tile_t_chunk=64)):
        announce("tile tiers", wtype, k, tune)
        prev = dawn.set_tuning(**tune)
        try:
            D = to_np(dawn.msssp(csr, srcs))
        finally:
            dawn.set_tuning(**prev)
        for j in (0, 1, k // 2, k - 1):
            assert_sssp_matches(g, int(srcs[j]), D[j], tag=f"{tune} col {j}")


@pytest.mark.parametrize("k", [33, 100, 200, 400])
def test_hop_count_pull_around_the_long_chunk_limit(dawn, k):
    # in-degrees around 64 (whole wavefront), its multiples and the chunk cuts
    g0 = _degree_graph([1, 2, 63, 64, 65, 128, 129, 255, 256, 257, 1023, 1024, 1025, 2100], "u32")
    rp = np.asarray(g0.rowptr)
    src = np.repeat(np.arange(g0.n), np.diff(rp))
    g = graphgen.from_edges(g0.n, np.asarray(g0.colidx), src, np.ones(g0.m, np.uint32), "u32")
    csr = dawn.Csr.from_graph(g)
    tg = dawn.tgraph(csr)
    srcs = np.random.default_rng(44).integers(0, g.n, k).astype(np.int32)
    for tune in (dict(tile_pull=0, tile_pull_src=0), dict()):
        announce("hop counts, long pull chunks", k, tune)
        prev = dawn.set_tuning(small_m=0, **tune)
        try:
            D = to_np(dawn.umsssp(csr, srcs, tgraph=tg)).view(np.uint32)
        finally:
            dawn.set_tuning(**prev)
        for j in (0, k // 2, k - 1):
            lv = oracle.bfs(g, int(srcs[j]))
            assert np.array_equal(D[j], np.where(lv < 0, 0xFFFFFFFF, lv).astype(np.uint32)), (tune, j)


@pytest.mark.parametrize("wtype", ["u32", "f32lognormal"])
@pytest.mark.parametrize("k", [28, 31, 32, 33, 64, 65, 200])
def test_steps_that_turn_from_push_to_pull_and_back(dawn, wtype, k):
    # frontiers that grow and shrink through the limits of the pull rule, with
    # fewer and more than half of a tile's columns live
    for g in (graphgen.er(40009, 320009, 51, weights=wtype), graphgen.rmat(14, 16, 52, weights=wtype)):
        csr = dawn.Csr.from_graph(g)
        tg = dawn.tgraph(csr)
        srcs = graphgen.pick_sources(g, k, 53)
        announce("push and pull by turns", g.name, k)
        prev = dawn.set_tuning(small_m=0)
        try:
            D = to_np(dawn.msssp(csr, srcs, tgraph=tg))
            P = to_np(dawn.msssp(csr, srcs))
        finally:
            dawn.set_tuning(**prev)
        assert np.array_equal(D.view(np.uint32), P.view(np.uint32))
        for j in (0, k - 1):
            assert_sssp_matches(g, int(srcs[j]), D[j], tag=f"{g.name} col {j}", check_invariants=False)
