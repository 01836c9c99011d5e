"""The tile's own tests and tuning lists with mode = 1, under which multi-source
calls take the tile whatever the graph's size: at the defaults most of their graphs
run in one workgroup per source or on copies, and the tile's tuning is not used.
Which of the two ran shows in the run info: only a tile reads an edge once for
several sources (union_edges < edges_scanned)."""
import numpy as np
import pytest

import graphgen
import test_gpu_autotune as autotune_tests
import test_gpu_batched as batched
import test_gpu_random_parity as random_parity
import test_gpu_tile_edge as tile_edge
import test_gpu_unweighted as unweighted
import test_gpu_wg_per_source as wg_per_source
from gpu_helpers import announce

pytestmark = pytest.mark.gpu


@pytest.fixture
def tile(dawn):
    prev = dawn.set_tuning(mode=1)
    yield dawn
    dawn.set_tuning(**prev)


@pytest.mark.parametrize("unit", [False, True])
def test_mode_1_takes_the_tile(dawn, unit):
    g = graphgen.rmat(13, 16, 21, weights="u32")
    csr = dawn.Csr.from_graph(g)
    srcs = graphgen.pick_sources(g, 152, 4)
    call = dawn.umsssp if unit else dawn.msssp
    for mode in (0, 1):
        announce("route", "hop counts" if unit else "weighted", "mode", mode)
        prev = dawn.set_tuning(mode=mode)
        try:
            info = dawn.info_tensor()
            call(csr, srcs, info=info)
        finally:
            dawn.set_tuning(**prev)
        i = dawn.read_info(info)
        assert (i["union_edges"] < i["edges_scanned"]) == (mode == 1)


@pytest.mark.parametrize("ti", range(len(batched.PULL_TUNINGS)))
@pytest.mark.parametrize("wk", ["u32", "f32lognormal"])
def test_pull_tunings(tile, wk, ti):
    batched.test_msssp_pull_steps_match_push_and_oracle(tile, wk, ti)


@pytest.mark.parametrize("wk", ["u32", "f32lognormal"])
def test_pull_quads(tile, wk):
    batched.test_msssp_pull_quads_of_four_and_one_segment(tile, wk)


def test_pull_hub_target(tile):
    batched.test_msssp_pull_hub_target_with_many_chunks(tile)


def test_pull_grid(tile):
    batched.test_msssp_pull_grid_f32_many_steps(tile)


def test_all_pairs(tile):
    batched.test_apsp_er_small_equals_floyd_warshall(tile)
    batched.test_apsp_f32_small(tile)


@pytest.mark.parametrize("pi", range(len(tile_edge.PATHS)))
@pytest.mark.parametrize("wt", ["u32", "f32"])
def test_edge_cases(tile, wt, pi):
    tile_edge.test_tile_edge_cases_match_oracle(tile, wt, pi)


@pytest.mark.parametrize("bad", ["n", "neg"])
def test_bad_source(tile, bad):
    tile_edge.test_msssp_bad_device_source_is_reported(tile, bad)


@pytest.mark.parametrize("ti", range(len(unweighted.PULL)))
def test_hop_counts(tile, ti):
    unweighted.test_umsssp_rmat_matches_bfs_and_weighted_unit(tile, ti)


@pytest.mark.parametrize("name", [
    "test_umsssp_counters_are_the_bfs_ones", "test_umsssp_five_segments",
    "test_umsssp_hub_target_with_many_chunks", "test_umsssp_grid_many_steps",
    "test_umsssp_chain_and_tiny_graphs", "test_umsssp_eight_segments",
    "test_unit_weight_type_batched_calls_are_hop_counts"])
def test_hop_count_shapes(tile, name):
    getattr(unweighted, name)(tile)


@pytest.mark.parametrize("i", range(random_parity.CASES))
def test_random_graphs(tile, i):
    random_parity.test_random_graph_sssp_and_msssp(tile, i)


@pytest.mark.parametrize("i", range(24))
def test_random_hop_counts(tile, i):
    random_parity.test_random_graph_hop_counts(tile, i)


def test_autotune(tile, tmp_path, monkeypatch):
    autotune_tests.test_autotune_keeps_results_and_caches(tile, tmp_path, monkeypatch)


# the tile's results where the library would take one workgroup per source
@pytest.mark.parametrize("wk", ["u32", "f32lognormal"])
@pytest.mark.parametrize("shape", wg_per_source.SHAPES)
def test_small_shapes(tile, shape, wk):
    wg_per_source.test_one_and_many_sources(tile, shape, wk)


# what the lists leave out: every random graph's tuning drawn once more, with pull
# steps at a drawn bound
@pytest.mark.parametrize("tj", range(len(random_parity.TILE_TUNINGS)))
@pytest.mark.parametrize("wk", ["u32", "f32lognormal"])
def test_tile_tunings_with_pull_steps(tile, wk, tj):
    from gpu_helpers import assert_sssp_matches, to_np
    g = graphgen.rmat(12, 16, 77, weights=wk)
    csr = tile.Csr.from_graph(g)
    tg = tile.tgraph(csr)
    srcs = graphgen.pick_sources(g, 130, 5)
    out = []
    for pull in (dict(tile_pull=100, tile_pull_src=2), dict(tile_pull=1001)):
        tune = dict(random_parity.TILE_TUNINGS[tj], **pull)
        announce("tile tunings with pull steps", wk, tune)
        prev = tile.set_tuning(**tune)
        try:
            out.append(to_np(tile.msssp(csr, srcs, tgraph=tg)))
        finally:
            tile.set_tuning(**prev)
    assert np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32))
    for j in (0, 64, 129):
        assert_sssp_matches(g, int(srcs[j]), out[0][j], tag=f"col {j}")
