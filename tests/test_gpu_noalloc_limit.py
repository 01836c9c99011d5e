"""The graphs that dawn_sssp_noalloc takes: exactly those whose two queues of n
ids, two queues of m / 65 + m / 256 + 2 records and three bitmaps, each rounded
up to 256 bytes, fit NOALLOC_SCRATCH_BYTES together with 2816 bytes."""
import ctypes

import numpy as np
import pytest

import graphgen
import paper_2306_07872_amd as dawn_mod
from gpu_helpers import announce, to_np


def _bytes(n, m):
    up = lambda x: (x + 255) // 256 * 256  # noqa: E731
    return 2816 + 2 * up(4 * n) + 2 * up(16 * (m // 65 + m // 256 + 2)) + 3 * up((n + 31) // 32 * 4)


def _limit(m):
    """The largest n whose graph of m edges is taken."""
    n = 1
    while _bytes(2 * n, m) <= dawn_mod.NOALLOC_SCRATCH_BYTES:
        n *= 2
    step = n
    while step:
        if _bytes(n + step, m) <= dawn_mod.NOALLOC_SCRATCH_BYTES:
            n += step
        step //= 2
    return n


@pytest.mark.parametrize("m", [0, 1000, 9_000_000, 60_000_000])
def test_larger_graphs_are_refused_on_the_host(m):
    lib = dawn_mod.load()
    n, fake, null = _limit(m) + 1, ctypes.c_void_p(0x1000), ctypes.c_void_p(0)
    assert lib.dawn_sssp_noalloc(fake, fake, fake, 0, n, m, 0, fake, null) == 3


@pytest.mark.gpu
@pytest.mark.parametrize("m", [1000, 9_000_000])
def test_the_largest_graph_is_taken(dawn, m):
    import torch
    n = _limit(m)
    rng = np.random.default_rng(m)
    src = np.sort(rng.integers(0, n, m)).astype(np.int64)
    src[: m // 2] = 5                       # a long row, in many records
    src.sort()
    dst = rng.integers(0, n, m)
    g = graphgen.from_edges(n, src, dst, rng.integers(1, 9, m).astype(np.uint32), "u32")
    csr = dawn.Csr.from_graph(g)
    for tune in (dict(), dict(mode=1, step_launches=3)):
        announce("noalloc at its limit", n, m, tune)
        prev = dawn.set_tuning(small_m=0, **tune)
        try:
            out = torch.full((n,), 7, dtype=torch.uint32, device="cuda")
            dawn.sssp_noalloc(csr, 5, out)
            ref = dawn.sssp(csr, 5)
        finally:
            dawn.set_tuning(**prev)
        assert np.array_equal(to_np(out), to_np(ref))
