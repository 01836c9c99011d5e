"""GPU parity of a single source whose row lies at a tier limit, on every launch
mix, with the device validation on and off, with a run info and without."""
import numpy as np
import pytest

import graphgen
from gpu_helpers import announce, assert_sssp_matches, to_np

pytestmark = pytest.mark.gpu

MIXES = [dict(), dict(mode=1, step_launches=2), dict(mode=1, step_launches=20), dict(mode=2, grid=3),
         dict(validate=1), dict(mode=1, step_launches=1, validate=1)]


@pytest.mark.parametrize("mi", range(len(MIXES)))
@pytest.mark.parametrize("deg", [0, 1, 8, 9, 64, 65, 96, 97, 256, 257, 1500])
def test_source_row_at_the_tier_limits(dawn, deg, mi):
    n, s = 3001, 2977
    rng = np.random.default_rng(deg)
    src = np.concatenate([np.full(deg, s), rng.integers(0, s, 6000)])
    dst = rng.integers(0, n, src.size)
    g = graphgen.from_edges(n, src, dst, rng.integers(1, 50, src.size).astype(np.uint32), "u32")
    csr = dawn.Csr.from_graph(g)
    prev = dawn.set_tuning(small_m=0, t_lane=8, t_wave=256, t_chunk=256, **MIXES[mi])
    try:
        announce("source row", deg, MIXES[mi])
        info = dawn.info_tensor()
        D = to_np(dawn.sssp(csr, s, info=info))
        assert dawn.read_info(info)["converged"] == 1
        P = to_np(dawn.sssp(csr, s))          # raises unless the run converged
    finally:
        dawn.set_tuning(**prev)
    assert_sssp_matches(g, s, D, tag=f"degree {deg} {MIXES[mi]}")
    assert np.array_equal(D, P)
