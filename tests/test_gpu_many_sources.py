"""More sources than one launch's workgroups may be (2^32 threads) on a small
graph: every row, the run info summed over the launches, a bad source."""
import numpy as np
import pytest

import graphgen
import oracle
from gpu_helpers import announce, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_k", [256, 320])
def test_four_million_sources(dawn, tile_k):
    import torch
    n, k = 7, (1 << 22) + 5
    g = graphgen.from_edges(n, [0, 1, 2, 3, 4, 0], [1, 2, 3, 4, 0, 5],
                            np.array([3, 1, 4, 1, 5, 9], np.uint32), "u32")
    csr = dawn.Csr.from_graph(g)
    ref = np.stack([oracle.sssp(g, s, "u32")[0] for s in range(n)])
    src = np.random.default_rng(1).integers(0, n, k).astype(np.int32)
    prev = dawn.set_tuning(tile_k=tile_k)
    try:
        announce("more sources than a launch holds", k, "tile_k", tile_k)
        info = dawn.info_tensor()
        D = to_np(dawn.msssp(csr, torch.as_tensor(src, device="cuda"), info=info)).view(np.uint32)
        i = dawn.read_info(info)
        assert np.array_equal(D, ref[src])
        reached = (ref != 0xFFFFFFFF).sum(axis=1)
        assert i["converged"] == 1 and i["improvements"] >= int((reached[src] - 1).sum())
        src[-1] = n
        with pytest.raises(dawn.DawnError):
            dawn.msssp(csr, torch.as_tensor(src, device="cuda"))
    finally:
        dawn.set_tuning(**prev)
