"""Batches whose graphs have weights of unlike scales: no graph waits for another,
so step t settles every vertex that a shortest path of t edges reaches: a run takes
at most the edges of the longest of the graphs' (shortest) shortest paths, and the
step that finds nothing."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import announce, to_np

pytestmark = pytest.mark.gpu


def _scaled(g, f):
    return g.with_weights((g.w.astype(np.float64) * f).astype(g.w.dtype), g.wtype)


def _run(dawn, gs, srcs, **tune):
    import torch
    b = dawn.Batch([dawn.Csr.from_graph(g) for g in gs])
    prev = dawn.set_tuning(**tune)
    try:
        info = dawn.info_tensor()
        out = b.run(torch.tensor(srcs, dtype=torch.int32, device="cuda"), info=info)
        parts = [to_np(x) for x in b.split(out)]
        return parts, dawn.read_info(info)
    finally:
        dawn.set_tuning(**prev)
        b.close()


@pytest.mark.parametrize("wk", ["f32lognormal", "u32"])
@pytest.mark.parametrize("case", ["persistent", "step launches", "one workgroup"])
def test_no_graph_waits_for_another(dawn, wk, case):
    n, m, cnt = (6000, 24000, 4) if case == "one workgroup" else (30000, 240000, 8)
    tune = {"persistent": dict(), "step launches": dict(mode=1, step_launches=8),
            "one workgroup": dict(small_m=1 << 20)}[case]
    base = [graphgen.er(n, m, 30 + i, **(dict(weights="u32", wlo=1, whi=200) if wk == "u32"
                                         else dict(weights=wk))) for i in range(cnt)]
    gs = [_scaled(g, 1000.0 if i == 1 else 1.0) for i, g in enumerate(base)]
    srcs = [int(graphgen.pick_sources(g, 1, 3)[0]) for g in gs]
    announce("unlike batch", wk, case)
    parts, info = _run(dawn, gs, srcs, **tune)
    assert info["converged"] == 1
    refs = [oracle.sssp(g, s, "u32" if g.wtype == "u32" else "f32fold") for g, s in zip(gs, srcs)]
    assert info["steps"] <= max(int(hops.max()) for _, hops in refs) + 1
    for (ref, _), d in zip(refs, parts):
        assert np.array_equal(d.view(np.uint32), ref.view(np.uint32))
