"""GPU parity of the fused 3D sweep over the tiles and z chunks it chooses by
the grid: sizes that are multiples of a tile (64 x 11, 32 x 16, 16 x 8) and of
a chunk, one more and one fewer, with and without a per-cell shear modulus.

Bars as for the other single sweeps: FP64 fields within 1e-11 and FP32 fields
within 2e-5 of the oracle (per field, stresses on the deviator scale), the
residual within 1e-9 / 1e-3.
"""
import numpy as np
import pytest

from ep_workloads import Model, random_state
from gpu_common import compare, it_names, say, set_state, solver
from oracle.oracle import Oracle

pytestmark = pytest.mark.gpu

GRIDS = [
    (16, 8, 6),        # one 16 x 8 tile, chunks of 3 planes
    (17, 9, 7),        # one cell more in every direction
    (64, 48, 30),      # whole 16 x 8 tiles with tiles strictly inside the domain
    (128, 128, 64),    # whole 32 x 16 tiles, chunks of 8 planes
    (127, 130, 67),
    (193, 122, 70),    # 16 x 8 tiles in chunks of 12 (FP32), 32 x 16 in chunks of 8 (FP64)
    (256, 132, 60),    # whole 64 x 11 tiles, chunks of 12 (FP32)
    (190, 127, 101),   # partial 64 x 11 tiles in chunks of 8 (FP32), 32 x 16 in chunks of 24 (FP64)
]


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
@pytest.mark.parametrize("with_g", [False, True], ids=["uniform", "G"])
@pytest.mark.parametrize("grid", GRIDS, ids=["x".join(map(str, g)) for g in GRIDS])
def test_fused_sweep_over_tiles_and_chunks(grid, with_g, prec):
    m = Model(ndim=3, nx=grid[0], ny=grid[1], nz=grid[2], ly=0.8, lz=0.6, incl_radius=0.2,
              shear=1.2 if with_g else 1.0)
    say("fused plan", grid, "G" if with_g else "uniform", "prec", prec)
    st = random_state(m, seed=5, amp_v=2e-3, amp_s=1.2e-3)
    g, o = solver(m, precision=prec, sweep=1), Oracle(m)
    if with_g:
        field = 1.2 * np.random.Generator(np.random.PCG64(3)).uniform(0.6, 1.0, m.n_cells)
        g.set_shear_modulus(field)
        o.set_shear_modulus(field)
    set_state(g, m, st, settable_tzz=False)
    set_state(o, m, st, settable_tzz=True)
    names = it_names(m)
    for _ in range(2):
        rg, ro = g.sweep(1), o.sweep()
        compare(m, g.fields(names), o.fields(names), names, 1e-11 if prec == 0 else 2e-5, str(grid))
        assert abs(rg - ro) <= (1e-9 if prec == 0 else 1e-3) * ro, (rg, ro)
    g.close()
