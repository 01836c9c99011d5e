"""A source outside [0, n) in a multi-source call ends the run of its tile_k
sources before its first step, on every route that the call may take: one
workgroup per source, copies of the graph, tiles.  The other tiles' rows, what
the failed tile's rows hold, and the count of failed runs are the tiles'."""
import numpy as np
import pytest

import graphgen
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu

# name, graph arguments, sources, positions of bad ones
CASES = [("edge-parallel", (900, 7001), 5, (1,)),
         ("edge-parallel, two bad", (900, 7001), 300, (3, 280)),
         ("bitmap scan", (20000, 100000), 7, (0, 6)),
         ("bitmap scan, second tile", (20000, 100000), 300, (299,)),
         ("copies", (50000, 300000), 5, (2,)),
         ("copies, two bad", (50000, 300000), 4, (0, 3))]


def _run(dawn, call, csr, srcs, **tune):
    import torch
    prev = dawn.set_tuning(**tune)
    try:
        info = dawn.info_tensor()
        D = to_np(call(csr, srcs, info=info, check=False))
        i = dawn.read_info(info)
        torch.cuda.synchronize()
        assert dawn.run_status() == (0, 1)
        call(csr, srcs, check=False)       # (msssp without info: the run-status record)
        torch.cuda.synchronize()
        return D, i, dawn.run_status()
    finally:
        dawn.set_tuning(**prev)


@pytest.mark.parametrize("unit", [False, True])
@pytest.mark.parametrize("ci", range(len(CASES)))
def test_bad_sources_end_their_tile(dawn, ci, unit):
    name, shape, k, bad = CASES[ci]
    g = graphgen.er(*shape, 2, weights="u32")
    csr = dawn.Csr.from_graph(g)
    srcs = graphgen.pick_sources(g, k, 3).astype(np.int32)
    for i, b in enumerate(bad):
        srcs[b] = (-1, g.n)[i % 2]
    call = dawn.umsssp if unit else dawn.msssp
    announce("bad sources", name, "hop counts" if unit else "weighted")
    D, i, status = _run(dawn, call, csr, srcs)
    T, ti, tstatus = _run(dawn, call, csr, srcs, mode=1)
    assert np.array_equal(D.view(np.uint32), T.view(np.uint32))
    assert i["converged"] == ti["converged"] == -1
    assert i["steps"] == ti["steps"] or not unit
    assert status == tstatus
    if not unit:
        failed = {b // 256 for b in bad}
        for j in (0, k - 1):
            if j // 256 not in failed:
                assert_sssp_matches(g, int(srcs[j]), D[j], tag=f"{name} row {j}", check_invariants=False)
