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
