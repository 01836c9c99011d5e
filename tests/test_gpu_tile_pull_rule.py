"""GPU parity of tile steps where the pull rule has no lower bound on the
frontier's edges (tile_pull = 0, or so few edges that the bound rounds to 0) but
does ask for active sources per edge: push steps, with more workgroups launched
than take part, mix with pull steps over many near-empty steps.  Every step is a
step launch on a graph large enough for the full push grid."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import INF32, announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu


def _levels(g, s):
    lv = oracle.bfs(g, int(s))
    return np.where(lv < 0, INF32, lv).astype(np.uint32)


def _run(dawn, call, csr, srcs, tg, **tune):
    prev = dawn.set_tuning(mode=1, **tune)   # mode 1: always the tile
    try:
        info = dawn.info_tensor()
        D = to_np(call(csr, srcs, info=info, tgraph=tg, check=False))
        return D, dawn.read_info(info)
    finally:
        dawn.set_tuning(**prev)


@pytest.mark.parametrize("pull_src", [16, 64])
@pytest.mark.parametrize("k", [40, 70])
def test_near_empty_steps(dawn, pull_src, k):
    for g in (graphgen.grid(260, 257, 0.01, 3, weights="u32"),
              graphgen.rmat(16, 8, 4, weights="f32lognormal")):
        csr = dawn.Csr.from_graph(g)
        tg = dawn.tgraph(csr)
        srcs = graphgen.pick_sources(g, k, 5)
        tune = dict(tile_pull=0, tile_pull_src=pull_src, tile_step_launches=4096)
        announce("pull rule without a bound, weighted", g.name, k, tune)
        D, info = _run(dawn, dawn.msssp, csr, srcs, tg, **tune)
        assert info["converged"] == 1
        for j in (0, k // 2, k - 1):
            assert_sssp_matches(g, int(srcs[j]), D[j], tag=f"{g.name} col {j}", check_invariants=False)
        announce("pull rule without a bound, hop counts", g.name, k, tune)
        D, info = _run(dawn, dawn.umsssp, csr, srcs, tg, **tune)
        assert info["converged"] == 1
        for j in (0, k // 2, k - 1):
            assert np.array_equal(D[j].view(np.uint32), _levels(g, srcs[j])), (g.name, j)
        assert info["steps"] == max(int(oracle.bfs(g, int(s)).max()) + 1 for s in srcs)


@pytest.mark.parametrize("m", [1, 2, 3, 9, 10])
def test_graphs_of_so_few_edges_that_the_bound_is_zero(dawn, m):
    # a path of m edges among isolated vertices, at the default pull bounds
    n = 70000
    g = graphgen.from_edges(n, np.arange(m), np.arange(1, m + 1), np.full(m, 3, np.uint32), "u32")
    csr = dawn.Csr.from_graph(g)
    tg = dawn.tgraph(csr)
    srcs = np.concatenate([np.zeros(40, np.int32), np.arange(30) % (m + 1)]).astype(np.int32)
    announce("few edges", m)
    D, info = _run(dawn, dawn.msssp, csr, srcs, tg)
    assert info["converged"] == 1 and info["steps"] == m + 1
    H, hinfo = _run(dawn, dawn.umsssp, csr, srcs, tg)
    assert hinfo["converged"] == 1 and hinfo["steps"] == m + 1
    for j in (0, 39, 40, 69):
        lv = _levels(g, srcs[j])
        assert np.array_equal(H[j].view(np.uint32), lv)
        assert np.array_equal(D[j].view(np.uint32), np.where(lv == INF32, INF32, 3 * lv))
