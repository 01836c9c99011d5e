"""Captured runs and the grid barrier.  barrier_ms = 0 gives up at the first wait
for another workgroup, so a captured run that still converges holds none."""
import numpy as np
import pytest

import graphgen
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu

# past the vertices that one workgroup's LDS holds, with at most small_m edges
SHAPES = [(32769, 40000), (60000, 120000), (131073, 131072)]


@pytest.mark.parametrize("wk", ["u32", "f32lognormal"])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_captured_runs_wait_for_no_other_workgroup(dawn, shape, wk):
    import torch
    g = graphgen.er(*shape, 5, weights=wk)
    csr = dawn.Csr.from_graph(g)
    s = int(graphgen.pick_sources(g, 1, 6)[0])
    ws = dawn.workspace(dawn.sssp_workspace_bytes(g.n, g.m))
    out = torch.empty(g.n, dtype=dawn.dist_dtype(g.wtype), device="cuda")
    info = dawn.info_tensor()
    dawn.sssp(csr, s, out=out, ws=ws, info=info)
    prev = dawn.set_tuning(barrier_ms=0)
    try:
        announce("captured small run", shape, wk)
        cg = torch.cuda.CUDAGraph()
        with torch.cuda.graph(cg):
            dawn.sssp(csr, s, out=out, ws=ws, info=info, check=False)
    finally:
        dawn.set_tuning(**prev)
    for rep in range(3):
        out.zero_()
        info.zero_()
        cg.replay()
        torch.cuda.synchronize()
        assert dawn.read_info(info)["converged"] == 1
        assert_sssp_matches(g, s, to_np(out), tag=f"replay {rep}", check_invariants=False)


def test_small_captured_batches_wait_for_no_other_workgroup(dawn):
    import torch
    gs = [graphgen.er(15000, 20000, 7 + i, weights="f32lognormal") for i in range(4)]
    b = dawn.Batch([dawn.Csr.from_graph(g) for g in gs])
    assert b.total_n > 32768 and b.total_m <= 131072
    srcs = [int(graphgen.pick_sources(g, 1, 8)[0]) for g in gs]
    src = torch.tensor(srcs, dtype=torch.int32, device="cuda")
    out = torch.empty(b.total_n, dtype=torch.float32, device="cuda")
    info = dawn.info_tensor()
    prev = dawn.set_tuning(barrier_ms=0)
    try:
        announce("captured small batch")
        b.capture(src, out, info=info)
    finally:
        dawn.set_tuning(**prev)
    for rep in range(3):
        out.zero_()
        b.replay()
        torch.cuda.synchronize()
        assert dawn.read_info(info)["converged"] == 1
        for g, s, d in zip(gs, srcs, b.split(out)):
            assert_sssp_matches(g, s, to_np(d), tag=f"replay {rep}", check_invariants=False)
    b.close()


@pytest.mark.parametrize("small", [False, True])
def test_batch_replays_on_two_streams(dawn, small):
    """A replay whose run holds a grid barrier waits for the one before it on
    another stream (held up here by a spin kernel); a one-workgroup run does not."""
    import torch
    n, m = (900, 4000) if small else (60000, 480000)
    g = graphgen.er(n, m, 9, weights="u32")
    csr = dawn.Csr.from_graph(g)
    s = int(graphgen.pick_sources(g, 1, 2)[0])
    src = torch.tensor([s], dtype=torch.int32, device="cuda")
    batches = [dawn.Batch([csr]) for _ in range(2)]
    outs = [torch.empty(n, dtype=torch.uint32, device="cuda") for _ in range(2)]
    for b, o in zip(batches, outs):
        b.capture(src, o)
        b.replay()
    torch.cuda.synchronize()
    for o in outs:
        o.fill_(7)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    ends = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    torch.cuda.synchronize()
    announce("batch replays on two streams", "small" if small else "large")
    with torch.cuda.stream(streams[0]):
        torch.cuda._sleep(200_000_000)
        batches[0].replay(stream=streams[0])
        ends[0].record()
    with torch.cuda.stream(streams[1]):
        batches[1].replay(stream=streams[1])
        ends[1].record()
    torch.cuda.synchronize()
    first = ends[0].elapsed_time(ends[1])   # ms from the first replay's end to the second's
    assert first < 0 if small else first > 0, first
    for b, o in zip(batches, outs):
        assert_sssp_matches(g, s, to_np(o), tag="two streams", check_invariants=False)
        b.close()
    dawn.check_runs()
