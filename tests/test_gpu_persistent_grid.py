"""Tuning fields of persistent single-source launches: `grid` is taken as given,
also above the size that the library would choose, and `coop` and `grid` serve
runs on copies of the graph."""
import time

import numpy as np
import pytest

import graphgen
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu


def _median_ms(call):
    import torch
    times = []
    for _ in range(7):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        call()
        torch.cuda.synchronize()
        times.append((time.perf_counter() - t0) * 1e3)
    return sorted(times)[3]


def test_grid_above_the_librarys_choice(dawn):
    """A path of 6000 steps, each little more than a barrier (1.9 us with 64
    workgroups, 3.3 us with 256): by itself the library takes 32 workgroups."""
    n = 6000
    g = graphgen.from_edges(n, np.arange(n - 1), np.arange(1, n), np.ones(n - 1, np.uint32), "u32")
    csr = dawn.Csr.from_graph(g)
    ms = {}
    for grid in (0, 32, 256):
        prev = dawn.set_tuning(small_m=0, grid=grid)
        try:
            announce("path, grid", grid)
            out = dawn.sssp(csr, 0)
            ms[grid] = _median_ms(lambda: dawn.sssp(csr, 0, out=out, check=False))
            dawn.check_runs()
        finally:
            dawn.set_tuning(**prev)
        assert np.array_equal(to_np(out).view(np.uint32), np.arange(n, dtype=np.uint32))
    assert ms[256] > 1.1 * ms[32] and ms[256] > 1.1 * ms[0], ms


@pytest.mark.parametrize("tune", [dict(coop=1), dict(grid=7), dict(grid=100000), dict(ss_tail_grid=3)])
def test_runs_under_launch_tunings(dawn, tune):
    g = graphgen.er(40009, 320009, 5, weights="f32lognormal")
    csr = dawn.Csr.from_graph(g)
    srcs = graphgen.pick_sources(g, 3, 6)
    prev = dawn.set_tuning(**tune)
    try:
        announce("launch tuning", tune)
        D = to_np(dawn.msssp(csr, srcs))
        d = to_np(dawn.sssp(csr, int(srcs[0])))
    finally:
        dawn.set_tuning(**prev)
    assert np.array_equal(D[0].view(np.uint32), d.view(np.uint32))
    for j in range(3):
        assert_sssp_matches(g, int(srcs[j]), D[j], tag=f"{tune} row {j}", check_invariants=False)
