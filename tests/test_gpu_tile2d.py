"""GPU parity of the 2D sweeps over the tile shapes that the library chooses by
the grid, and of launches that do several sweeps: windows of sweeps shorter
and longer than a launch holds, on grids that are a multiple of a tile, one
cell more and one fewer, with and without a per-cell shear modulus.

Bars as for the other single sweeps: FP64 fields within 1e-11 and FP32 fields
within 2e-5 of the oracle (per field, stresses on the deviator scale), the
residual within 1e-9 / 1e-3.  A window of sweeps in one call equals the same
sweeps one by one bit for bit.
"""
import numpy as np
import pytest

from ep_workloads import Model, random_state
from gpu_common import compare, it_names, say, set_state, solver
from oracle.oracle import Oracle

pytestmark = pytest.mark.gpu

# tiles per direction reach one and two workgroups per CU (256 CUs) of the
# 12 x 12, 16 x 16, 20 x 20, 24 x 24, 32 x 32 and 52 x 20 shapes
GRIDS = [(12, 12), (13, 11), (24, 36), (192, 192), (193, 191), (256, 256), (257, 255), (320, 320), (321, 319),
         (440, 400), (520, 500), (640, 641), (777, 500), (1024, 1024)]


def pair(grid, with_g, prec, seed=7):
    m = Model(ndim=2, nx=grid[0], ny=grid[1], ly=0.9, incl_radius=0.2, shear=1.2 if with_g else 1.0)
    st = random_state(m, seed=seed, amp_v=2e-3, amp_s=1.2e-3)
    g, o = solver(m, precision=prec), Oracle(m)
    if with_g:
        field = 1.2 * np.random.Generator(np.random.PCG64(3)).uniform(0.6, 1.0, m.n_cells)
        g.set_shear_modulus(field)
        o.set_shear_modulus(field)
    set_state(g, m, st, settable_tzz=False)
    set_state(o, m, st, settable_tzz=True)
    return m, g, o


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("with_g", [False, True], ids=["uniform", "G"])
@pytest.mark.parametrize("grid", GRIDS, ids=["x".join(map(str, g)) for g in GRIDS])
def test_tile_shapes_match_oracle(grid, with_g, prec):
    say("2d tiles", grid, "G" if with_g else "uniform", "prec", prec)
    m, g, o = pair(grid, with_g, prec)
    names = it_names(m)
    for n in (1, 3, 6):
        rg = g.sweep(n)
        for _ in range(n):
            ro = o.sweep()
        compare(m, g.fields(names), o.fields(names), names, 1e-11 if prec == 0 else 2e-5, f"{grid} {n}")
        assert abs(rg - ro) <= (1e-9 if prec == 0 else 1e-3) * ro, (n, rg, ro)
    g.close()


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("grid", [(63, 63), (250, 240), (383, 191), (500, 490), (1000, 300)],
                         ids=lambda g: "x".join(map(str, g)))
def test_windows_of_sweeps_equal_single_sweeps(grid, prec):
    m, a, o = pair(grid, False, prec)
    _, b, _ = pair(grid, False, prec)
    ra = a.sweep(23)
    for _ in range(23):
        rb = b.sweep(1)
    assert ra == rb
    for n in it_names(m):
        assert np.array_equal(a.get(n), b.get(n)), n
    a.close()
    b.close()
