"""Persistent launches whose grid barriers give up at once (barrier_ms = 0) while
workgroups of the same launch are still starting: every kernel exits, every run
is reported, and the next run with the normal bound is right.  Every row is
queued (t_lane = 1) and the grid is as large as the device holds."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import INF32, announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu

# call, sources, tuning that reaches its persistent launch
CASES = {
    "sssp": (1, dict(small_m=0, mode=2, t_lane=1, t_wave=64)),
    "copies": (4, dict(small_m=0, t_lane=1, t_wave=64)),
    "msssp": (70, dict(mode=2)),
    "umsssp": (70, dict(mode=2)),
}


@pytest.mark.parametrize("what", sorted(CASES))
def test_runs_that_give_up_while_workgroups_start(dawn, what):
    k, tune = CASES[what]
    g = graphgen.er(300000, 2400000, 3, weights="u32")
    csr = dawn.Csr.from_graph(g)
    srcs = graphgen.pick_sources(g, k, 4)

    def run(info):
        if what == "sssp":
            return dawn.sssp(csr, int(srcs[0]), info=info, check=False)
        call = dawn.umsssp if what == "umsssp" else dawn.msssp
        return call(csr, srcs, info=info, check=False)

    prev = dawn.set_tuning(barrier_ms=0, **tune)
    try:
        for rep in range(10):
            announce("give-up while starting", what, rep)
            info = dawn.info_tensor()
            run(info)
            assert dawn.read_info(info)["converged"] == -2
        dawn.set_tuning(barrier_ms=prev["barrier_ms"])
        info = dawn.info_tensor()
        D = to_np(run(info)).reshape(k, g.n)
        assert dawn.read_info(info)["converged"] == 1
    finally:
        dawn.set_tuning(**prev)
    s = int(srcs[-1])
    if what == "umsssp":
        lv = oracle.bfs(g, s)
        assert np.array_equal(D[-1].view(np.uint32), np.where(lv < 0, INF32, lv).astype(np.uint32))
    else:
        assert_sssp_matches(g, s, D[-1], tag=what, check_invariants=False)
