"""Rules that choose how a sweep is launched (host code only, no GPU): the
tile and chunk length of the fused 3D sweep by the grid."""
import ctypes as C
import os

import pytest

WIDE, SQUARE, SMALL = 0, 1, 2      # tiles of the fused 3D sweep: 64 x 11, 32 x 16, 16 x 8


@pytest.fixture(scope="module")
def lib():
    import torch  # noqa: F401  (its HIP runtime, before the library binds to another)
    from paper_2305_01701_amd import ep
    if not os.path.exists(ep.LIB_PATH):
        from paper_2305_01701_amd import build
        build.build()
    return C.CDLL(ep.LIB_PATH)


def plan_3d(lib, fp32, with_g, nx, ny, nz):
    """(tile, planes per chunk) that ep::fused_plan_3d gives for a grid."""
    f = lib._ZN2ep13fused_plan_3dEbbiiil
    f.restype = C.c_uint64
    sy = (nx + 1 + 31) // 32 * 32
    r = f(C.c_bool(fp32), C.c_bool(with_g), nx, ny, nz, C.c_long(sy * (ny + 1)))
    return r & 0xffffffff, r >> 32


@pytest.mark.parametrize("with_g", [False, True], ids=["uniform", "G"])
@pytest.mark.parametrize("nz", [3, 4, 6, 8])
def test_slabs_that_fill_the_chip_take_no_small_tiles(lib, nz, with_g):
    """500 x 500 FP32 slabs: 2016 small tiles fill the chip and are bound by
    their halo's bytes (8 planes: 79 us against 63 with 32 x 16 tiles)."""
    assert plan_3d(lib, True, with_g, 500, 500, nz)[0] == SQUARE


def test_small_grids_take_small_tiles(lib):
    assert plan_3d(lib, True, False, 63, 63, 63) == (SMALL, 4)
    assert plan_3d(lib, True, False, 300, 300, 5)[0] == SMALL
    assert plan_3d(lib, False, False, 63, 63, 63) == (SMALL, 4)


@pytest.mark.parametrize("fp32,grid", [(False, (4959, 4950, 3)), (False, (4959, 4950, 8)), (True, (7200, 7100, 5))])
def test_long_planes_keep_the_fused_sweep(lib, fp32, grid):
    """Planes of which no chunk fits into 2 GiB (FP64 4959 x 4950: 196 MB)
    run in the fused sweep, on its 32 x 16 tiles."""
    tile, zc = plan_3d(lib, fp32, False, *grid)
    assert tile == SQUARE and zc >= 3


def test_planes_beyond_2_gib_are_out_of_range(lib):
    assert plan_3d(lib, False, False, 20000, 20000, 3)[1] == 0


def one_sweep(lib, fp32, nx, ny):
    f = lib._ZN2ep16tile2d_one_sweepEblli
    f.restype = C.c_int
    tiles = lambda y: C.c_long(-(-nx // 60) * -(-ny // y))
    return f(C.c_bool(fp32), tiles(12), tiles(28), 256)


def test_single_2d_sweeps_take_tiles_without_a_wide_halo(lib):
    """One sweep per launch: 60 x 12 tiles (10), 60 x 28 (11) where they spare
    the CUs a second workgroup or, in FP32, rounds of workgroups."""
    for fp32 in (False, True):
        assert one_sweep(lib, fp32, 63, 63) == 10 and one_sweep(lib, fp32, 700, 700) == 10
        assert one_sweep(lib, fp32, 511, 511) == 11 and one_sweep(lib, fp32, 2047, 2047) == 10
    assert one_sweep(lib, True, 1023, 1023) == 11 and one_sweep(lib, False, 1023, 1023) == 10


@pytest.mark.parametrize("fp32", [False, True], ids=["fp64", "fp32"])
def test_workspace_holds_no_field_for_transfers(lib, fp32):
    """3D: 46 FP64 fields (two sets of 9 iterates, 6 increment-start ones,
    cohesion, Lambda, compliance, start velocities, displacements, strains, 4
    diagnostics, guess), with FP32 iterates 27 more in FP32; the array that
    packs a field for the host is one of them."""
    from ep_workloads import c3_3d
    from paper_2305_01701_amd import ep
    m = c3_3d()
    nelem = (m.nx + 1 + 31) // 32 * 32 * (m.ny + 1) * (m.nz + 1)
    fields = 46 * 8 + (27 * 4 if fp32 else 0)
    ws = ep.ep_workspace_size(ep.params_from_model(m, precision=ep.EP_FP32_FIELDS if fp32 else ep.EP_FP64))
    assert fields * nelem <= ws <= fields * nelem + 75 * 256 + 4096


@pytest.mark.parametrize("reps,sweeps", [(1, 6), (3, 6), (5, 6), (6, 6), (7, 12), (100, 102), (2 ** 31 - 1, 2 ** 31 - 2)])
def test_the_tuner_times_the_sweeps_it_is_asked_for(lib, reps, sweeps):
    """Rounded up to whole launches of shapes with two and with three sweeps."""
    assert lib._ZN2ep12tuned_sweepsEi(reps) == sweeps


def common_shape(lib, fp32, own, tiles, scale=None, own_scale=1.0):
    f = lib._ZN2ep13tile2d_commonEbPKlS1_PKddi
    f.restype = C.c_int
    arr = lambda d: (C.c_long * 10)(*[d.get(s, 0) for s in range(10)])
    sc = (C.c_double * 10)(*[(scale or {}).get(s, 1.0) for s in range(10)])
    return f(C.c_bool(fp32), arr(own), arr(tiles), sc, C.c_double(own_scale), 256)


@pytest.mark.parametrize("fp32", [False, True], ids=["fp64", "fp32"])
def test_tuned_shapes_give_way_only_to_the_tuners_own_times(lib, fp32):
    """Three models of 63 x 63 cells: the shapes for few tiles are modelled faster
    than shape 0; where the tuner measured them slower than the shapes it chose,
    these stay, and where it measured 16 x 16 tiles (7) as the fastest, all
    models take those."""
    cells = {0: (52, 20) if fp32 else (56, 8), 6: (12, 12), 7: (16, 16), 8: (20, 20), 9: (32, 32) if fp32 else (20, 20)}
    tiles = {s: 3 * -(-63 // x) * -(-63 // y) for s, (x, y) in cells.items()}
    own = {0: tiles[0]}
    assert common_shape(lib, fp32, own, tiles) in (6, 7, 8)
    slow = {s: 3.0 for s in (6, 7, 8, 9)}
    assert common_shape(lib, fp32, own, tiles, slow, 0.5) == -1
    assert common_shape(lib, fp32, own, tiles, {6: 3.0, 7: 0.1, 8: 3.0, 9: 3.0}) == 7
    assert common_shape(lib, fp32, own, tiles, own_scale=0.0) == -1
