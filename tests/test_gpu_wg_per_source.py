"""GPU parity of the one-workgroup kernels that hold a run's state in LDS: the
edge-parallel kernel (4, 8 or 16 edges per thread), the bitmap-scan kernel (its
three sizes, and one vertex past the largest), each for one source and as one
workgroup per source of a multi-source call.  Distances are unique, so every
result equals the oracle bit for bit."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu

# (n, m): edge-parallel instances and their limits, then the bitmap-scan sizes
SHAPES = [(1, 0), (2, 1), (33, 100), (700, 4096), (700, 4097), (1531, 8192), (1531, 8193),
          (6144, 16384), (6144, 16385), (6145, 9000), (16384, 70001), (16385, 50000),
          (32768, 131072), (32769, 40000)]


def _graph(n, m, wk):
    if m == 0:
        return graphgen.from_edges(n, [], [], np.zeros(0, np.uint32 if wk == "u32" else np.float32),
                                   "u32" if wk == "u32" else "f32")
    return graphgen.er(n, m, 5 * n + m, weights=wk)


@pytest.mark.parametrize("wk", ["u32", "f32lognormal"])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_and_many_sources(dawn, shape, wk):
    n, m = shape
    g = _graph(n, m, wk)
    csr = dawn.Csr.from_graph(g)
    rng = np.random.default_rng(n + m)
    for k in (1, 5):
        srcs = rng.integers(0, n, k).astype(np.int32)
        srcs[-1] = n - 1
        announce("workgroup per source", shape, wk, "k", k)
        info = dawn.info_tensor()
        D = to_np(dawn.msssp(csr, srcs, info=info))
        assert dawn.read_info(info)["converged"] == 1
        lone = to_np(dawn.sssp(csr, int(srcs[0])))
        assert np.array_equal(D[0].view(np.uint32), lone.view(np.uint32))
        for j in range(k):
            assert_sssp_matches(g, int(srcs[j]), D[j], tag=f"{shape} {wk} col {j}")


def test_long_rows_span_edge_windows(dawn):
    """Hub rows of many times the edges that are marked at a time, next to
    rows of one edge and rows without edges."""
    n = 20000
    hub = np.arange(1, n)
    src = np.concatenate([np.zeros(n - 1, np.int64), hub[::3], np.full(3000, 7)])
    dst = np.concatenate([hub, (hub[::3] * 5) % n, np.arange(9000, 12000)])
    w = np.random.default_rng(4).integers(1, 1000, src.size).astype(np.uint32)
    g = graphgen.from_edges(n, src, dst, w, "u32")
    csr = dawn.Csr.from_graph(g)
    srcs = np.array([0, 7, 4, 2, 19999], np.int32)
    announce("hub rows in one workgroup")
    D = to_np(dawn.msssp(csr, srcs))
    for j, s in enumerate(srcs):
        assert_sssp_matches(g, int(s), D[j], tag=f"hub col {j}")


@pytest.mark.parametrize("n,m", [(900, 7001), (5000, 60000), (20000, 100000)])
def test_hop_counts_and_counters(dawn, n, m):
    """Unit weights: levels, and the counters of sequential Algorithm 2 summed
    over the sources."""
    g = graphgen.er(n, m, n, weights="u32one")
    csr = dawn.Csr.from_graph(g)
    srcs = graphgen.pick_sources(g, 6, 3)
    lv = [oracle.bfs(g, int(s)) for s in srcs]
    for run in (dawn.umsssp, dawn.msssp):
        announce("hop counts, workgroup per source", n, m, run.__name__)
        info = dawn.info_tensor()
        D = to_np(run(csr, srcs, info=info)).view(np.uint32)
        i = dawn.read_info(info)
        for j in range(len(srcs)):
            assert np.array_equal(D[j], np.where(lv[j] < 0, 0xFFFFFFFF, lv[j]).astype(np.uint32))
        assert i["converged"] == 1
        assert i["steps"] == max(int(x.max()) + 1 for x in lv)
        assert i["edges_scanned"] == sum(oracle.m_reach(g, int(s)) for s in srcs)
        assert i["improvements"] == sum(int((x >= 0).sum()) - 1 for x in lv)


@pytest.mark.parametrize("n,m", [(900, 7001), (20000, 100000)])
def test_source_out_of_range_is_reported(dawn, n, m):
    g = graphgen.er(n, m, 2)
    csr = dawn.Csr.from_graph(g)
    for bad in (-1, n):
        announce("bad source", n, bad)
        with pytest.raises(dawn.DawnError) as e:
            dawn.msssp(csr, np.array([3, bad, 5], np.int32))
        assert e.value.status == dawn.E_INCOMPLETE and "-1" in str(e.value)
        info = dawn.info_tensor()
        dawn.msssp(csr, np.array([3, bad, 5], np.int32), info=info, check=False)
        assert dawn.read_info(info)["converged"] == -1


@pytest.mark.parametrize("wk", ["u32", "f32unit"])
def test_far_rows_wait(dawn, wk):
    """Even graphs with enough edges that steps leave far rows for later."""
    for g in (graphgen.er(9001, 70001, 3, weights=wk), graphgen.grid(150, 151, 0.01, 5, weights=wk),
              graphgen.er(32768, 131072, 4, weights=wk)):
        csr = dawn.Csr.from_graph(g)
        srcs = graphgen.pick_sources(g, 3, 8)
        announce("workgroup per source, far rows", g.name, wk)
        D = to_np(dawn.msssp(csr, srcs))
        for j, s in enumerate(srcs):
            assert_sssp_matches(g, int(s), D[j], tag=f"{g.name} {wk} col {j}")
            assert np.array_equal(to_np(dawn.sssp(csr, int(s))).view(np.uint32), D[j].view(np.uint32))
