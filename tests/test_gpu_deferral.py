"""GPU parity of single-source runs that leave far frontier rows for later steps:
every launch mix, every row tier (tiny thresholds send ordinary rows through
the queued tiers), weights from zero to the type's limits.  Distances are
unique, so every result equals the oracle bit for bit; at unit weights nothing
is deferred and the counters are sequential Algorithm 2's."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu

TUNINGS = [
    dict(small_m=0),
    dict(small_m=0, t_lane=2, t_wave=64, t_chunk=256),         # rows queued, few hubs in chunks
    dict(small_m=0, t_lane=1, t_wave=64, grid=3, wg_threads=256),
    dict(small_m=0, mode=1, step_launches=6),                  # state handed to the persistent launch
    dict(small_m=0, mode=1, step_launches=4096, t_lane=2, t_wave=64),
    dict(small_m=0, ss_skip=0),
    dict(small_m=0, grid=1),
]


def _run(dawn, g, s, **tune):
    import torch
    prev = dawn.set_tuning(**tune)
    try:
        info = dawn.info_tensor()
        out = dawn.sssp(dawn.Csr.from_graph(g), int(s), info=info)
        torch.cuda.synchronize()
        return to_np(out), dawn.read_info(info)
    finally:
        dawn.set_tuning(**prev)


def _check(dawn, g, s, tag, **tune):
    announce("deferral", tag, "n", g.n, "m", g.m, "source", int(s), tune)
    d, info = _run(dawn, g, s, **tune)
    assert_sssp_matches(g, int(s), d, tag=f"{tag} {tune}")
    assert info["converged"] == 1 and info["steps"] <= g.n


@pytest.mark.parametrize("ti", range(len(TUNINGS)))
def test_even_graphs_match_oracle(dawn, ti):
    for g in (graphgen.grid(173, 211, 0.01, 3, weights="f32unit"),
              graphgen.grid(64, 700, 0.0, 4, weights="u32"),
              graphgen.er(20011, 160077, 5, weights="f32lognormal"),
              graphgen.er(20011, 160077, 6, weights="u32", wlo=1, whi=100000)):
        _check(dawn, g, graphgen.pick_sources(g, 1, ti)[0], g.name, **TUNINGS[ti])


def test_long_rows_in_an_even_graph(dawn):
    """Rows of 300 and 5000 edges (wave and chunk tiers at the default
    thresholds) among rows of 8: few enough not to switch deferral off."""
    g0 = graphgen.er(60000, 480000, 8, weights="u32", wlo=1, whi=1000)
    src = np.repeat(np.arange(g0.n), g0.outdeg()).astype(np.int64)
    rng = np.random.default_rng(9)
    hs = np.concatenate([np.full(5000, 17), np.repeat(rng.integers(0, g0.n, 40), 300)])
    src = np.concatenate([src, hs])
    dst = np.concatenate([g0.colidx.astype(np.int64), rng.integers(0, g0.n, hs.size)])
    w = np.concatenate([g0.w, rng.integers(1, 1000, hs.size).astype(np.uint32)])
    g = graphgen.from_edges(g0.n, src, dst, w, "u32")
    for tune in (dict(small_m=0), dict(small_m=0, mode=1, step_launches=5),
                 dict(small_m=0, t_wave=256, t_chunk=256)):
        for s in (17, 5, int(hs[-1])):
            _check(dawn, g, s, "long rows", **tune)


@pytest.mark.parametrize("lo,hi", [(0, 0), (0, 1), (1, 2), (0, 3_000_000_000), (2**31, 2**32 - 2)])
def test_weight_ranges_u32(dawn, lo, hi):
    """Zero weights, and sums that saturate."""
    g0 = graphgen.er(9000, 70001, 7, weights="u32")
    w = np.random.default_rng(lo % 1000 + hi % 1000).integers(lo, hi + 1, g0.m).astype(np.uint32)
    g = g0.with_weights(w, "u32")
    for tune in (TUNINGS[0], TUNINGS[3]):
        _check(dawn, g, 3, f"weights {lo}..{hi}", **tune)


@pytest.mark.parametrize("scale", [0.0, 1e-42, 1e-30, 1e30])
def test_weight_ranges_f32(dawn, scale):
    """Zeros, denormals, and large weights."""
    g0 = graphgen.er(9000, 70001, 8, weights="f32lognormal")
    g = g0.with_weights((g0.w * np.float32(scale)).astype(np.float32), "f32")
    for tune in (TUNINGS[0], TUNINGS[4]):
        announce("deferral f32 scale", scale, tune)
        d, info = _run(dawn, g, 3, **tune)
        d32, _ = oracle.sssp(g, 3, "f32fold")
        assert np.array_equal(np.asarray(d).view(np.uint32), d32.view(np.uint32))
        assert info["converged"] == 1


@pytest.mark.parametrize("ti", range(len(TUNINGS)))
def test_unit_weight_counters(dawn, ti):
    for g in (graphgen.grid(150, 130, 0.01, 3, weights="f32one"),
              graphgen.er(20011, 160077, 5, weights="u32one")):
        s = int(graphgen.pick_sources(g, 1, 2)[0])
        announce("deferral, unit weights", g.name, TUNINGS[ti])
        d, info = _run(dawn, g, s, **TUNINGS[ti])
        _, c = oracle.govm(g, s)
        for key in ("steps", "edges_scanned", "improvements", "frontier_entries"):
            assert info[key] == c[key], key


def test_graphs_of_unlike_scales_in_one_batch(dawn):
    """One threshold serves all graphs of a batch."""
    import torch
    gs = [graphgen.grid(90, 90, 0.01, 1, weights="f32unit"),
          graphgen.er(30000, 240000, 2, weights="f32lognormal")]
    gs.append(gs[1].with_weights(gs[1].w * np.float32(1e4), "f32"))
    gs.append(gs[0].with_weights(gs[0].w * np.float32(1e-4), "f32"))
    srcs = [5, 77, 77, 4000]
    for tune in (dict(small_m=0), dict(small_m=0, mode=1, step_launches=9)):
        announce("deferral, batch", tune)
        prev = dawn.set_tuning(**tune)
        try:
            b = dawn.Batch([dawn.Csr.from_graph(g) for g in gs])
            out = b.run(torch.tensor(srcs, dtype=torch.int32, device="cuda"))
            dawn.check_runs()
            for g, s, d in zip(gs, srcs, b.split(out)):
                d32, _ = oracle.sssp(g, s, "f32fold")
                assert np.array_equal(to_np(d).view(np.uint32), d32.view(np.uint32))
            b.close()
        finally:
            dawn.set_tuning(**prev)
