"""GPU parity of multi-source calls of a few sources, which run as one
single-source run on copies of the graph: copies that straddle bitmap words,
queued rows (tiny thresholds), repeated sources, sources without out-edges, the
workspace entry points, HIP-graph replay, bad sources."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu

TUNINGS = [dict(small_m=0),
           dict(small_m=0, t_lane=2, t_wave=64, t_chunk=256),
           dict(small_m=0, t_lane=1, t_wave=64, grid=2, wg_threads=256),
           dict(small_m=0, ss_skip=0)]


def _graphs():
    # vertex counts that are and are not multiples of 32
    yield graphgen.grid(37, 41, 0.01, 3, weights="f32unit"), 9
    yield graphgen.grid(64, 64, 0.02, 4, weights="u32"), 3
    yield graphgen.er(5003, 40009, 5, weights="u32", wlo=0, whi=50), 7
    yield graphgen.er(1024, 8000, 6, weights="f32lognormal"), 2
    yield graphgen.rmat(12, 16, 7, weights="u32"), 8


@pytest.mark.parametrize("ti", range(len(TUNINGS)))
def test_copies_match_oracle(dawn, ti):
    prev = dawn.set_tuning(**TUNINGS[ti])
    try:
        for g, k in _graphs():
            csr = dawn.Csr.from_graph(g)
            srcs = np.random.default_rng(ti + k).integers(0, g.n, k).astype(np.int32)
            srcs[0], srcs[-1] = g.n - 1, srcs[k // 2]
            announce("copies", g.name, "k", k, TUNINGS[ti])
            info = dawn.info_tensor()
            D = to_np(dawn.msssp(csr, srcs, info=info))
            assert dawn.read_info(info)["converged"] == 1
            for j in range(k):
                assert_sssp_matches(g, int(srcs[j]), D[j], tag=f"{g.name} col {j}")
    finally:
        dawn.set_tuning(**prev)


@pytest.mark.parametrize("ti", range(len(TUNINGS)))
def test_hop_counts_and_counters(dawn, ti):
    prev = dawn.set_tuning(**TUNINGS[ti])
    try:
        for g, k in ((graphgen.grid(45, 37, 0.01, 8, weights="u32one"), 6),
                     (graphgen.rmat(12, 16, 9, weights="u32one"), 3)):
            csr = dawn.Csr.from_graph(g)
            srcs = graphgen.pick_sources(g, k, 5)
            lv = [oracle.bfs(g, int(s)) for s in srcs]
            for run in (dawn.umsssp, dawn.msssp):
                announce("copies, hop counts", g.name, TUNINGS[ti], run.__name__)
                info = dawn.info_tensor()
                D = to_np(run(csr, srcs, info=info)).view(np.uint32)
                i = dawn.read_info(info)
                for j in range(k):
                    assert np.array_equal(D[j], np.where(lv[j] < 0, 0xFFFFFFFF, lv[j]).astype(np.uint32))
                assert i["steps"] == max(int(x.max()) + 1 for x in lv)
                assert i["edges_scanned"] == sum(oracle.m_reach(g, int(s)) for s in srcs)
                assert i["improvements"] == sum(int((x >= 0).sum()) - 1 for x in lv)
    finally:
        dawn.set_tuning(**prev)


def test_workspace_reverse_graph_and_replay(dawn):
    """The workspace that the tile would take serves, with and without a
    reverse graph, and a captured call replays with new sources."""
    import torch
    g = graphgen.grid(211, 307, 0.01, 11, weights="f32unit")   # past the one-workgroup sizes
    csr = dawn.Csr.from_graph(g)
    tg = dawn.tgraph(csr)
    k = 5
    src_t = torch.as_tensor(graphgen.pick_sources(g, k, 1), dtype=torch.int32, device="cuda")
    out = torch.empty((k, g.n), dtype=torch.float32, device="cuda")
    ws = dawn.workspace(dawn.msssp_workspace_bytes(g.n, g.m, k))
    info = dawn.info_tensor()
    announce("copies, replay")
    dawn.msssp(csr, src_t, out=out, ws=ws, info=info, tgraph=tg)
    s = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        dawn.msssp(csr, src_t, out=out, ws=ws, info=info, check=False)
    for rep in range(3):
        new = graphgen.pick_sources(g, k, 20 + rep)
        src_t.copy_(torch.as_tensor(new, dtype=torch.int32))
        graph.replay()
        torch.cuda.synchronize()
        got = to_np(out).copy()
        assert dawn.read_info(info)["converged"] == 1
        eager = to_np(dawn.msssp(csr, new, ws=ws, info=info, tgraph=tg))
        assert np.array_equal(got.view(np.uint32), eager.view(np.uint32))
        assert_sssp_matches(g, int(new[2]), got[2], tag=f"replay {rep}", check_invariants=False)


def test_source_out_of_range_is_reported(dawn):
    g = graphgen.er(50000, 300000, 2)
    csr = dawn.Csr.from_graph(g)
    for bad in (-1, g.n):
        announce("copies, bad source", bad)
        with pytest.raises(dawn.DawnError) as e:
            dawn.msssp(csr, np.array([3, bad, 5], np.int32))
        assert e.value.status == dawn.E_INCOMPLETE and "-1" in str(e.value)


def test_persistent_runs_on_two_streams(dawn):
    """Single-source and few-source runs whose launches hold a grid barrier, put
    on two streams by turns with nothing ordering them: all converge."""
    import torch
    g = graphgen.grid(300, 301, 0.01, 12, weights="f32unit")
    h = graphgen.rmat(15, 16, 13, weights="u32")
    cg, ch = dawn.Csr.from_graph(g), dawn.Csr.from_graph(h)
    sg, sh = graphgen.pick_sources(g, 4, 2), graphgen.pick_sources(h, 4, 3)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    src = [torch.as_tensor(x[:3].copy(), dtype=torch.int32, device="cuda") for x in (sg, sh)]
    ws = [dawn.workspace(dawn.msssp_workspace_bytes(c.n, c.m, 3)) for c in (cg, ch)]
    out = [torch.empty((3, c.n), dtype=dawn.dist_dtype(c.wtype), device="cuda") for c in (cg, ch)]
    one = [torch.empty(c.n, dtype=dawn.dist_dtype(c.wtype), device="cuda") for c in (cg, ch)]
    torch.cuda.synchronize()
    announce("two streams of persistent runs")
    for rep in range(6):
        for i, (c, s) in enumerate(((cg, sg), (ch, sh))):
            with torch.cuda.stream(streams[i]):
                dawn.msssp(c, src[i], out=out[i], ws=ws[i], stream=streams[i], check=False)
                dawn.sssp(c, int(s[3]), out=one[i], stream=streams[i], check=False)
    torch.cuda.synchronize()
    assert dawn.run_status() == (0, 1)
    for i, (gr, s) in enumerate(((g, sg), (h, sh))):
        for j in range(3):
            assert_sssp_matches(gr, int(s[j]), to_np(out[i])[j], tag="two streams", check_invariants=False)
        assert_sssp_matches(gr, int(s[3]), to_np(one[i]), tag="two streams", check_invariants=False)
