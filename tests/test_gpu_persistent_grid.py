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


def _star(n, wtype):
    """A hub (vertex 0) with an edge to every other vertex and one back from each."""
    w = np.random.default_rng(n).integers(1, 99, 2 * (n - 1))
    src = np.concatenate([np.zeros(n - 1, np.int64), np.arange(1, n)])
    dst = np.concatenate([np.arange(1, n), np.zeros(n - 1, np.int64)])
    dt = {"u32": np.uint32, "f32": np.float32, "i32": np.int32}[wtype]
    return graphgen.from_edges(n, src, dst, w.astype(dt), wtype), w[: n - 1]


@pytest.mark.parametrize("wtype", ["u32", "f32", "i32", "unit"])
@pytest.mark.parametrize("n", [2000, 196609, 196610, 524289, 524290])
def test_uneven_rows_around_the_size_limits(dawn, n, wtype):
    """2 (n - 1) edges: below and from 3 << 17 and 1 << 20 on."""
    g, w = _star(n, "u32" if wtype == "unit" else wtype)
    csr = dawn.Csr.from_graph(g, wtype="unit") if wtype == "unit" else dawn.Csr.from_graph(g)
    announce("star", n, wtype)
    prev = dawn.set_tuning(small_m=0)
    try:
        info = dawn.info_tensor()
        d = to_np(dawn.sssp(csr, 0, info=info))
        leaf = to_np(dawn.sssp(csr, n - 1))
    finally:
        dawn.set_tuning(**prev)
    i = dawn.read_info(info)
    # the hub's edges, the leaves' edges back, and every leaf lowered once
    assert i["converged"] == 1 and i["steps"] == 2
    assert i["edges_scanned"] == g.m and i["improvements"] == n - 1
    one = np.ones(n - 1) if wtype == "unit" else w
    assert d[0] == 0 and np.array_equal(d[1:].astype(np.int64), one.astype(np.int64))
    assert leaf[n - 1] == 0 and leaf[0] == (1 if wtype == "unit" else np.asarray(g.w)[-1])


def test_uneven_rows_take_the_whole_device(dawn):
    """Two edges per vertex, but two steps of two million edges: 882 us with 32
    workgroups, 240 with 256."""
    g, w = _star(2_000_000, "u32")
    csr = dawn.Csr.from_graph(g)
    ms = {}
    for grid in (0, 256):
        prev = dawn.set_tuning(grid=grid)
        try:
            announce("wide star, grid", grid)
            out = dawn.sssp(csr, 0)
            ms[grid] = _median_ms(lambda: dawn.sssp(csr, 0, out=out, check=False))
            dawn.check_runs()
        finally:
            dawn.set_tuning(**prev)
    assert np.array_equal(to_np(out)[1:].astype(np.int64), w)
    assert ms[0] < 1.5 * ms[256], ms
