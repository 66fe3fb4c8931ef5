"""Every form of the fused 3D sweep on the tiles of large grids (32 x 16 in both
precisions, 64 x 11 in FP32; the grids here are the small ones that choose
them): update sweeps with each option of the return, physical evaluations,
storing Lambda and sweeps with the held one, and slabs whose one chunk starts at
plane 0 and ends at the top.

Bars as for the other single sweeps: FP64 fields within 1e-11 and FP32 fields
within 2e-5 of the oracle, residual norms within 1e-9; whole FP64 increments
with equal iteration counts and fields within 1e-6.  The residuals of FP32
sweeps at the checks: within 1e-3 and three times the rounding floor that the
solver assumes for them, 8 u32 max|sigma| / h."""
import numpy as np
import pytest

from ep_workloads import Model, gaussian_shear, random_state
from gpu_common import compare, it_names, say, set_state, solver
from oracle.oracle import Oracle
from test_launch_plans import SQUARE, WIDE, lib, plan_3d  # noqa: F401

pytestmark = pytest.mark.gpu

FP64, FP32 = 0, 1
FORMS = [((129, 66, 40), FP64, SQUARE), ((129, 66, 40), FP32, SQUARE), ((228, 65, 40), FP32, WIDE)]
IDS = ["32x16-fp64", "32x16-fp32", "64x11-fp32"]
OPTIONS = {"plain": {}, "psi": dict(psi_deg=10.0), "eta_vp": dict(eta_vp=1e-3), "blend": dict(pt_blend=0.0),
           "all": dict(psi_deg=8.0, eta_vp=1e-3, shear=1.2)}


def pair(m, prec, with_g, seed):
    st = random_state(m, seed=seed, amp_v=2e-3, amp_s=1.2e-3)
    g, o = solver(m, precision=prec, sweep=1), Oracle(m)
    if with_g:
        G = gaussian_shear(m, centre=(0.03, -0.02, 0.01))
        g.set_shear_modulus(G)
        o.set_shear_modulus(G)
    set_state(g, m, st, settable_tzz=False)
    set_state(o, m, st, settable_tzz=True)
    return g, o


@pytest.mark.parametrize("name", OPTIONS)
@pytest.mark.parametrize("grid,prec,tile", FORMS, ids=IDS)
def test_update_sweeps_with_options(lib, grid, prec, tile, name):
    with_g = name == "all" and tile == SQUARE      # no 64 x 11 tiles with a per-cell G
    assert plan_3d(lib, prec == FP32, with_g, *grid)[0] == tile
    m = Model(ndim=3, nx=grid[0], ny=grid[1], nz=grid[2], ly=0.5, lz=0.3, c0=1e-4, incl_radius=0.1, **OPTIONS[name])
    say("update sweeps", grid, "prec", prec, name)
    g, o = pair(m, prec, with_g, 23)
    names = it_names(m)
    for n in (3, 2):
        g.sweep(n)
        for _ in range(n):
            o.sweep()
        compare(m, g.fields(names), o.fields(names), names, 1e-11 if prec == FP64 else 2e-5, name)
    g.close()
    o.close()


@pytest.mark.parametrize("with_g", [False, True], ids=["uniform", "G"])
@pytest.mark.parametrize("grid", [(129, 66, 40), (127, 130, 67)], ids=lambda g: "x".join(map(str, g)))
def test_physical_evaluation(lib, grid, with_g):
    assert plan_3d(lib, False, with_g, *grid)[0] == SQUARE
    m = Model(ndim=3, nx=grid[0], ny=grid[1], nz=grid[2], ly=0.5, lz=0.3, c0=1e-4, psi_deg=8.0, eta_vp=1e-3,
              shear=1.2 if with_g else 1.0)
    say("physical evaluation", grid, with_g)
    g, o = pair(m, FP64, with_g, 29)
    r = g.residual()
    assert r["physical"] == pytest.approx(o.sweep(physical=True), rel=1e-9)
    assert r["resid"] == pytest.approx(o.evaluate(), rel=1e-9)
    g.close()
    o.close()


def frozen_model(grid, **kw):
    return Model(ndim=3, nx=grid[0], ny=grid[1], nz=grid[2], ly=0.5, lz=0.3, dt=6e-4, n_check=10, incl_radius=0.1,
                 incl_centre=(0.04, -0.03, 0.02), eta_vp=5e-5, psi_deg=5.0, freeze_iter=40, **kw)


def test_increments_with_frozen_plasticity_match_oracle(lib):
    m = frozen_model((129, 66, 40), tol=2e-2, max_iter=3000)
    assert plan_3d(lib, False, False, m.nx, m.ny, m.nz)[0] == SQUARE
    g, o = solver(m, precision=FP64, sweep=1), Oracle(m)
    for n in range(2):
        sg, so = g.load_step(), o.load_step()
        say("frozen increment", n, sg["iters"], sg["frozen_at"], sg["n_yield"])
        assert sg["status"] == 0 and so["status"] == 0
        assert sg["frozen_at"] == so["frozen_at"] == 40 and sg["n_yield"] == so["n_yield"] > 1000
        assert sg["iters"] == so["iters"] > 60
    names = it_names(m) + ["eps_p"]
    compare(m, g.fields(names), o.fields(names), it_names(m), 1e-6)
    assert np.abs(g.get("eps_p") - o.get("eps_p")).max() <= 1e-6 * np.abs(o.get("eps_p")).max()
    g.close()
    o.close()


@pytest.mark.parametrize("grid,tile", [((129, 66, 40), SQUARE), ((228, 65, 40), WIDE)], ids=["32x16", "64x11"])
def test_fp32_checks_before_and_after_the_freeze(lib, grid, tile):
    assert plan_3d(lib, True, False, *grid)[0] == tile
    m = frozen_model(grid, tol=1e-9, max_iter=120)
    g, o = solver(m, precision=FP32, sweep=1), Oracle(m)
    o.record_history()
    sg, so = g.load_step(), o.load_step()
    hg, pg = g.history()
    ho = o.history() / so["ref"]
    assert sg["frozen_at"] == so["frozen_at"] == 40 and list(pg) == [FP32] * 12 and len(ho) == 12
    # stresses of the elastic predictor bound those of the increment
    sigma = 2.0 * (m.bulk + m.shear) * m.dt
    floor = 8.0 * 5.96e-8 * sigma / min(m.lx / m.nx, m.ly / m.ny, m.lz / m.nz) / so["ref"]
    say("fp32 checks", grid, floor, [(float(a), float(b)) for a, b in zip(hg, ho)])
    for a, b in zip(hg, ho):
        assert abs(a - b) <= 1e-3 * b + 3.0 * floor, (a, b, floor)
    g.close()
    o.close()


@pytest.mark.parametrize("prec", [FP64, FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("with_g", [False, True], ids=["uniform", "G"])
@pytest.mark.parametrize("grid", [(500, 70, 3), (300, 300, 3), (40, 30, 4)], ids=lambda g: "x".join(map(str, g)))
def test_slabs(grid, with_g, prec):
    m = Model(ndim=3, nx=grid[0], ny=grid[1], nz=grid[2], ly=0.8, lz=0.1, c0=1e-4, incl_radius=0.05,
              shear=1.2 if with_g else 1.0)
    say("slab", grid, with_g, prec)
    g, o = pair(m, prec, with_g, 31)
    names = it_names(m)
    for n in (1, 3):
        rg = g.sweep(n)
        for _ in range(n):
            ro = o.sweep()
        compare(m, g.fields(names), o.fields(names), names, 1e-11 if prec == FP64 else 2e-5, str(grid))
        assert abs(rg - ro) <= (1e-9 if prec == FP64 else 1e-3) * ro
    g.close()
    o.close()
