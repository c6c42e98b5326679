"""The sizes on which the GPU tests of the large-tile GEMMs run do reach the tiles they name: the rules of
tile_rule.hpp, compiled for the host, evaluated for the 256 CUs of an MI355X.  A change of a rule that empties
one of those tests fails here."""
import ctypes
import os
import shutil
import subprocess

import pytest

import test_gpu_phase_gemm as phase

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_18631_amd", "csrc")
CUS = 256
TILES = ["64x128", "128x256", "256x128", "256x256", "320x256"]
SWIGLU, BF16, SCATTER = range(3)

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("rule") / "rule.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", CSRC,
                    os.path.join(HERE, "tile_rule.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    i, l = ctypes.c_int, ctypes.c_long
    lib.fwd_tile.argtypes = [i, i, i, l, l, l, i]
    lib.bwd_rows_tile.argtypes = [i, l, l, l, i, i]
    lib.wgrad_on_ring.argtypes = [l, l]
    return lib


@pytest.mark.parametrize("case", phase.SEGMENTS, ids=str)
def test_segment_cases_reach_their_tiles(rule, case):
    """moe_grouped_ffn passes the capacity per local expert as the expected rows."""
    rows, d, F, up, down = case
    E = len(phase.COUNTS)
    assert TILES[rule.fwd_tile(CUS, F, d, E, rows, 0, SWIGLU)] == up
    assert TILES[rule.fwd_tile(CUS, d, F, E, rows, 0, BF16)] == down


def test_segment_cases_cover_both_schedules():
    """Each tile height with one, two, three and more K slices, with and without a partial last one."""
    slices = lambda K: (min(-(-K // 64), 4), K % 64 != 0)
    up = {(c[3], *slices(c[1])) for c in phase.SEGMENTS}
    down = {(c[4], *slices(c[2])) for c in phase.SEGMENTS}
    for n in (1, 2, 3, 4):
        for tail in (False, True):
            for tile in ("256x256", "320x256"):
                assert (tile, n, tail) in up and (tile, n, tail) in down, (tile, n, tail)


def test_few_tile_cases_reach_the_small_tile(rule):
    for T, d, F in phase.FEW_TILES:
        assert TILES[rule.fwd_tile(CUS, F, d, 1, T, 0, SWIGLU)] == "64x128"
        assert TILES[rule.fwd_tile(CUS, d, F, 1, T, 0, BF16)] == "64x128"


def test_backward_cases_reach_their_tiles(rule):
    E = len(phase.BACKWARD_COUNTS)
    for rows, d, F, tile in phase.BACKWARD:
        assert TILES[rule.bwd_rows_tile(CUS, E, rows, rows * E, d, 2 * F)] == tile


def test_a_partial_slice_keeps_the_tile(rule):
    """The forward's tile follows from the tile counts; a K that is no multiple of 64 does not change it."""
    for E, rows, N in [(32, 256, 2048), (32, 290, 6384), (64, 227, 3184), (8, 569, 6408), (64, 400, 1000)]:
        for epilogue in (SWIGLU, BF16):
            tiles = {TILES[rule.fwd_tile(CUS, N, K, E, rows, 0, epilogue)] for K in (2040, 2048, 2056)}
            assert len(tiles) == 1, (E, rows, N, epilogue, tiles)
    assert TILES[rule.fwd_tile(CUS, 2040, 2040, 32, 256, 0, BF16)] == "320x256"


def test_short_weight_gradients_stay_on_the_ring_kernel(rule):
    """One and two K slices: except for a handful of rows into whole lines."""
    for rows in (1, 16, 32):
        assert not rule.wgrad_on_ring(rows, 2560) and rule.wgrad_on_ring(rows, 2528) and rule.wgrad_on_ring(rows, 2552)
    for rows in (33, 64, 100, 128):
        assert all(rule.wgrad_on_ring(rows, pitch) for pitch in (2560, 2528, 2552))
    for rows in (0, 129, 256, 4000):
        assert not any(rule.wgrad_on_ring(rows, pitch) for pitch in (2560, 2528, 2552))


def test_short_backward_cases_reach_both_kernels(rule):
    on_ring = {(bool(rule.wgrad_on_ring(rows, d)), d % 64 == 0) for rows, d, F in phase.SHORT}
    assert on_ring == {(False, True), (True, True), (True, False)}


@pytest.mark.parametrize("tm, tn", [(1, 1), (2, 56), (3, 14), (56, 16), (7, 1)])
def test_weight_gradient_orders(rule, tm, tn):
    """Each visits every tile once; the router's m-fastest, the others n-fastest."""
    mn = (ctypes.c_int * 2)()
    for f32 in (0, 1):
        seen = []
        for i in range(tm * tn):
            rule.wgrad_order(i, tm, tn, f32, mn)
            seen.append((mn[0], mn[1]))
        assert seen == ([(m, n) for n in range(tn) for m in range(tm)] if f32 else
                        [(m, n) for m in range(tm) for n in range(tn)])


def test_bands_of_small_tiles_hold_a_shared_experts_rows(rule):
    """Launches on 64- and 128-row tiles share their weights with a dense extra group of up to 512 rows; its weights are
    streamed once per band."""
    assert rule.band_m(64) * 64 >= 512 and rule.band_m(128) * 128 >= 512
    assert rule.band_m(256) == rule.band_m(320) == 4
