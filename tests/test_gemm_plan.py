"""Host logic of the bf16 GEMM's launch schedule: tile coverage of every grid the library would build (no GPU)."""
import itertools

import pytest

from paper_2603_13289_amd import binding as rc
from tests import test_gpu_gemm_whole_calls as whole_calls
from tests import test_gpu_qkv_rope as qkv_rope


def test_every_tile_is_covered_exactly_once_on_the_workload_shapes():
    shapes = [(m, n, k, swiglu) for m in (33, 256, 1024, 1025, 1088, 1089, 1639, 3687, 5120, 7373, 36864)
              for (n, k, swiglu) in ((6144, 4096, False), (4096, 4096, False), (14336, 4096, True), (4096, 14336, False),
                                     (27648, 5120, True), (5120, 27648, False), (7168, 5120, False))]
    for (m, n, k, swiglu), tile, ws in itertools.product(shapes, (5, 6, 7), (True, False)):
        if tile == 7 and (swiglu or n % 192):
            continue
        err, nb = rc.rc_gemm_plan_check(m, n, k, swiglu, tile, 256, ws)
        assert err == 0, (m, n, k, swiglu, tile, ws, nb)
        assert nb > 0


@pytest.mark.parametrize("n_cus", [256, 304, 64, 8])
def test_coverage_over_a_sweep_of_row_counts(n_cus):
    """All row counts around the tile and round boundaries, ragged last tile rows of every height."""
    for n, k, swiglu in ((2048, 256, False), (16384, 128, False), (8192, 64, True), (384, 1024, False)):
        for m in list(range(1, 600)) + list(range(1000, 1300, 7)) + [4095, 4096, 4097, 4160, 4161]:
            for tile in (5, 6, 7):
                if tile == 7 and (swiglu or n % 192):
                    continue
                err, _ = rc.rc_gemm_plan_check(m, n, k, swiglu, tile, n_cus, True)
                assert err == 0, (m, n, k, swiglu, tile, n_cus)


@pytest.mark.parametrize("tile", [0, 8, 9, 10, 11, 12, 13])
def test_every_tile_type_covers_the_output_and_fits_the_workspace(tile):
    """The tile types that share one K partition: at 193 to 256 rows, 192-row tiles cut in 16 parts would hold half as
    much again as the workspace does."""
    rows = (1, 33, 61, 64, 65, 100, 192, 193, 200, 256, 257, 400, 449, 600, 1025, 1639, 2500, 5120)
    shapes = ((6144, 4096), (4096, 4096), (1024, 4096), (4096, 14336), (7168, 5120), (5120, 27648), (777, 448))
    for m, (n, k), swiglu, ws in itertools.product(rows, shapes, (False, True), (True, False)):
        assert rc.rc_gemm_plan_check(m, n, k, swiglu, tile, 256, ws)[0] == 0, (m, n, k, swiglu, ws)
    for n_cus, m in itertools.product((8, 64, 304), range(1, 420, 19)):
        assert rc.rc_gemm_plan_check(m, 768, 1024, False, tile, n_cus, True)[0] == 0, (n_cus, m)


def test_thin_tiles_are_used_for_a_one_row_remainder():
    """1024 + 1 rows against a wide N: the schedule with the thin last tile row needs fewer workgroups than
    five full tile rows would."""
    rc.rc_tune_set(rc.RC_TUNE_GEMM_THIN_TILES, 0)
    try:
        err0, nb_plain = rc.rc_gemm_plan_check(1025, 14336, 4096, True, 5, 256, True)
    finally:
        rc.rc_tune_set(rc.RC_TUNE_GEMM_THIN_TILES, 1)
    err1, nb_thin = rc.rc_gemm_plan_check(1025, 14336, 4096, True, 5, 256, True)
    assert err0 == 0 and err1 == 0
    assert nb_thin != nb_plain


def test_coverage_without_the_xcd_regrouping():
    rc.rc_tune_set(rc.RC_TUNE_GEMM_XCD_REMAP, 0)
    try:
        for m in (1, 255, 257, 1025, 1088, 1639, 5120):
            for (n, k, swiglu) in ((6144, 4096, False), (14336, 4096, True), (4096, 14336, False)):
                for tile in (5, 6, 7):
                    if tile == 7 and (swiglu or n % 192):
                        continue
                    assert rc.rc_gemm_plan_check(m, n, k, swiglu, tile, 256, True)[0] == 0, (m, n, k, tile)
    finally:
        rc.rc_tune_set(rc.RC_TUNE_GEMM_XCD_REMAP, 1)


def test_bad_arguments():
    assert rc.rc_gemm_plan_check(0, 64, 64, False, 5)[0] == -1
    assert rc.rc_gemm_plan_check(64, 64, 100, False, 5)[0] == -1
    assert rc.rc_gemm_plan_check(64, 64, 64, False, 4)[0] == -1


def test_coverage_of_the_schedules_the_library_chooses():
    """Tile type by shape, among them a thin last tile row behind whole tiles."""
    for n, k, swiglu in ((28672 // 2, 4096, True), (16384, 128, False), (4096, 14336, False), (6144, 4096, False), (5120, 27648, False)):
        for m in list(range(33, 700, 31)) + [768, 769, 1024, 1025, 1088, 1089, 1639, 2050, 2112, 2113, 5121]:
            for ws in (True, False):
                err, nb = rc.rc_gemm_plan_check(m, n, k, swiglu, 0, 256, ws)
                assert err == 0 and nb > 0, (m, n, k, swiglu, ws)


def _blocks(m, n, k, swiglu, workspace, thin=1):
    rc.rc_tune_set(rc.RC_TUNE_GEMM_THIN_TILES, thin)
    try:
        return rc.rc_gemm_plan_check(m, n, k, swiglu, 0, 256, workspace)[1]
    finally:
        rc.rc_tune_set(rc.RC_TUNE_GEMM_THIN_TILES, 1)


@pytest.mark.parametrize("m,n,k,epilogue,workspace", [(*c, True) for c in whole_calls.THIN] + [(*c, False) for c in whole_calls.THIN_WHOLE])
def test_shapes_that_take_the_thin_body(m, n, k, epilogue, workspace):
    swiglu = epilogue == "swiglu"
    tiles = -(-m // 256) * -(-n // (128 if swiglu else 256))
    assert _blocks(m, n, k, swiglu, workspace) == -(-tiles // 8) * 8 != _blocks(m, n, k, swiglu, workspace, thin=0)


def test_shapes_of_few_rows_that_are_cut_in_parts():
    most = 0
    for m, n, k, epilogue in whole_calls.FEW:
        swiglu = epilogue == "swiglu"
        blocks, tiles = _blocks(m, n, k, swiglu, True), -(-n // (64 if swiglu else 128))   # tiles of 64 rows by 128 weight rows
        assert k % 256 and n % 16 == 0 and blocks != _blocks(m, n, k, swiglu, False)
        assert blocks % tiles == 0 and 4 <= blocks // tiles <= 16, (m, n, k)
        most = max(most, blocks // tiles * (2 if swiglu else 1) * (2 if m > 16 else 1))
    assert most == 64   # accumulator tiles of 1 KB: all the LDS that a launch gets without asking


@pytest.mark.parametrize("m,d,nq,nkv,page,tile", qkv_rope.THIN)
def test_shapes_of_qkv_with_a_thin_row_and_cut_tiles(m, d, nq, nkv, page, tile):
    n = (nq + 2 * nkv) * 128
    blocks = _blocks(m, n, d, False, True)
    assert blocks != _blocks(m, n, d, False, True, thin=0)      # thin tiles, which are never cut
    assert blocks > -(-(-(-m // 256) * -(-n // 256)) // 8) * 8  # more workgroups than tiles: others are
