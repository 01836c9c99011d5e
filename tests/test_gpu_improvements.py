"""The improvements counter where rows wait: per step, the vertices that the step
lowered, each once.  In the graph here every count is fixed whatever the order:
a chain takes one step per vertex, and every chain vertex lowers a few far
targets, which wait in the frontier while they are lowered again."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu

L, T = 400, 6


def _far_targets(wk):
    """Vertices 0..L a chain of weight 1, L+1..L+T the targets, the rest a part
    that no source reaches and whose small weights keep the threshold low."""
    n = 30000
    c = np.arange(L + 1)
    src = [c[:-1], np.repeat(c, T)]
    dst = [c[1:], np.tile(np.arange(L + 1, L + 1 + T), L + 1)]
    w = [np.ones(L), np.repeat(100000 - 10 * c, T)]
    rest = np.arange(L + 1 + T, n)
    for d in range(1, 8):
        src.append(rest)
        dst.append(L + 1 + T + (rest - (L + 1 + T) + d) % rest.size)
        w.append(np.ones(rest.size))
    dt = np.uint32 if wk == "u32" else np.float32
    return graphgen.from_edges(n, np.concatenate(src), np.concatenate(dst),
                               np.concatenate(w).astype(dt), wk)


TUNINGS = [
    dict(small_m=0),
    dict(small_m=0, grid=3, wg_threads=256),
    dict(small_m=0, t_lane=6, t_wave=64),              # the chain's rows queued, the targets scanned
    dict(small_m=0, mode=1, step_launches=50),
    dict(small_m=0, mode=1, step_launches=4096),
    dict(small_m=0, mode=1, step_launches=50, ss_pull=500),   # a pull-capable launch that pushes
    dict(small_m=0, mode=1, step_launches=4096, ss_pull=0),   # and one that pulls
]


@pytest.mark.parametrize("wk", ["u32", "f32"])
@pytest.mark.parametrize("ti", range(len(TUNINGS)))
def test_lowered_while_waiting(dawn, ti, wk):
    g = _far_targets(wk)
    csr = dawn.Csr.from_graph(g)
    tg = dawn.tgraph(csr) if "ss_pull" in TUNINGS[ti] else None
    announce("improvements", wk, TUNINGS[ti])
    prev = dawn.set_tuning(**TUNINGS[ti])
    try:
        info = dawn.info_tensor()
        d = to_np(dawn.sssp(csr, 0, info=info, tgraph=tg))
    finally:
        dawn.set_tuning(**prev)
    i = dawn.read_info(info)
    _, c = oracle.govm(g, 0)
    assert c["improvements"] == L + T * (L + 1)
    assert i["improvements"] == c["improvements"]
    assert_sssp_matches(g, 0, d, tag="far targets")


def test_copies_and_batches(dawn):
    import torch
    g = _far_targets("u32")
    csr = dawn.Csr.from_graph(g)
    prev = dawn.set_tuning(small_m=0)
    try:
        announce("improvements, copies")
        info = dawn.info_tensor()
        dawn.msssp(csr, np.array([0, 0, L + 1], np.int32), info=info)
        assert dawn.read_info(info)["improvements"] == 2 * (L + T * (L + 1))
        announce("improvements, batch")
        b = dawn.Batch([csr, csr])
        info = dawn.info_tensor()
        b.run(torch.tensor([0, L + 1], dtype=torch.int32, device="cuda"), info=info)
        torch.cuda.synchronize()
        assert dawn.read_info(info)["improvements"] == L + T * (L + 1)
        b.close()
    finally:
        dawn.set_tuning(**prev)


def test_never_below_the_reached_vertices(dawn):
    """Ordinary even graphs: at least one lowering for each vertex reached."""
    for g in (graphgen.er(40009, 320009, 5, weights="f32lognormal"),
              graphgen.grid(300, 301, 0.01, 6, weights="f32unit")):
        csr = dawn.Csr.from_graph(g)
        tg = dawn.tgraph(csr)
        s = int(graphgen.pick_sources(g, 1, 7)[0])
        for tune, t in ((dict(small_m=0), None), (dict(small_m=0, mode=1, step_launches=30), None),
                        (dict(small_m=0, mode=1, ss_pull=100), tg)):
            announce("improvements, bound", g.name, tune)
            prev = dawn.set_tuning(**tune)
            try:
                info = dawn.info_tensor()
                d = to_np(dawn.sssp(csr, s, info=info, tgraph=t))
            finally:
                dawn.set_tuning(**prev)
            assert dawn.read_info(info)["improvements"] >= int(np.isfinite(d).sum()) - 1


@pytest.mark.parametrize("threads", [0, 256])
@pytest.mark.parametrize("wk", ["u32", "f32"])
def test_lowered_while_waiting_in_one_workgroup(dawn, wk, threads):
    g = _far_targets(wk)
    csr = dawn.Csr.from_graph(g)
    prev = dawn.set_tuning(small_m=1 << 20, wg_threads=threads)
    try:
        announce("improvements, one workgroup", wk, threads)
        info = dawn.info_tensor()
        assert_sssp_matches(g, 0, to_np(dawn.sssp(csr, 0, info=info)), tag="one workgroup")
        assert dawn.read_info(info)["improvements"] == L + T * (L + 1)
        info = dawn.info_tensor()
        D = to_np(dawn.msssp(csr, np.array([0, L + 1, 0], np.int32), info=info))
        assert_sssp_matches(g, 0, D[2], tag="workgroup per source")
        assert dawn.read_info(info)["improvements"] == 2 * (L + T * (L + 1))
    finally:
        dawn.set_tuning(**prev)


@pytest.mark.parametrize("mids", [700, 8000])
def test_lowered_many_times_in_one_step(dawn, mids):
    """A source, `mids` vertices at descending distances, and two targets that each
    of them lowers, all in one step: the targets count once.  The edge-parallel and
    the bitmap-scan kernel, alone and per source, against the tile."""
    a = np.arange(1, mids + 1)
    src = np.concatenate([np.zeros(mids, np.int64), a, a])
    dst = np.concatenate([a, np.full(mids, mids + 1), np.full(mids, mids + 2)])
    w = np.concatenate([2 * mids - a, np.full(2 * mids, 5)]).astype(np.uint32)
    g = graphgen.from_edges(mids + 3, src, dst, w, "u32")
    csr = dawn.Csr.from_graph(g)
    announce("improvements, many decreases", mids)
    info = dawn.info_tensor()
    dawn.sssp(csr, 0, info=info)
    assert dawn.read_info(info)["improvements"] == mids + 2
    for tune in (dict(), dict(mode=1)):
        prev = dawn.set_tuning(**tune)
        try:
            info = dawn.info_tensor()
            dawn.msssp(csr, np.array([0, 3, 0], np.int32), info=info)
        finally:
            dawn.set_tuning(**prev)
        assert dawn.read_info(info)["improvements"] == 2 * (mids + 2) + 2, tune
def test_counted_up_to_the_step_limit(dawn):
    """A negative cycle in one workgroup: n steps, each lowering one vertex of the
    ring that the source leads into."""


STEP_LIMIT_TUNINGS = [dict(), dict(small_m=0), dict(small_m=0, mode=1, step_launches=10),
                      dict(small_m=0, mode=1, step_launches=4096),
                      dict(small_m=0, mode=1, step_launches=4096, ss_pull=0)]


@pytest.mark.parametrize("ti", range(len(STEP_LIMIT_TUNINGS)))
def test_counted_up_to_the_step_limit(dawn, ti):
    """A negative cycle: n steps, each lowering one vertex of the ring that the
    source leads into, the last one among them."""
    tune = STEP_LIMIT_TUNINGS[ti]
    ring = 70
    src = np.concatenate([[0], np.arange(1, ring + 1)])
    dst = np.concatenate([[1], np.arange(1, ring + 1) % ring + 1])
    g = graphgen.from_edges(ring + 1, src, dst, np.full(ring + 1, -1, np.int32), "i32")
    csr = dawn.Csr.from_graph(g)
    tg = dawn.tgraph(csr) if "ss_pull" in tune else None
    announce("improvements, step limit", tune)
    prev = dawn.set_tuning(**tune)
    try:
        info = dawn.info_tensor()
        dawn.sssp(csr, 0, info=info, tgraph=tg, check=False)
        i = dawn.read_info(info)
    finally:
        dawn.set_tuning(**prev)
    assert i["converged"] == 0 and i["steps"] == g.n
    assert i["improvements"] == g.n
