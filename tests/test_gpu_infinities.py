"""Infinities inside a fused 2D sweep: a cell whose two velocity gradients are
finite and whose divergence overflows gives the stresses, at its vertices too,
and the non-finite entries of the unfused kernels."""
import numpy as np
import pytest

from ep_workloads import Model
from gpu_common import IT2, say, solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_overflowing_divergence(prec):
    from paper_2305_01701_amd import ep
    m = Model(ndim=2, nx=40, ny=40, lx=40.0, ly=40.0)            # spacing 1: gradients are differences
    big = 0.6 * (np.finfo(np.float64).max if prec == 0 else float(np.finfo(np.float32).max))
    got = {}
    for form in (ep.EP_SWEEP_UNFUSED, ep.EP_SWEEP_FUSED):
        g = solver(m, precision=prec, sweep=form)
        vx, vy = g.get("vx").reshape(40, 41), g.get("vy").reshape(41, 40)
        vx[20, 18:] = big                                        # dvx of cell (17, 20)
        vy[21:, 17] = big                                        # dvy of cell (17, 20)
        g.set("vx", vx)
        g.set("vy", vy)
        g.sweep(1)
        got[form] = g.fields(IT2)
        g.close()
    a, b = got[ep.EP_SWEEP_UNFUSED], got[ep.EP_SWEEP_FUSED]
    say("infinities", prec, {k: int((~np.isfinite(a[k])).sum()) for k in IT2})
    assert any((~np.isfinite(a[k])).any() for k in IT2)
    for k in IT2:
        f = np.isfinite(a[k])
        assert np.array_equal(np.isnan(a[k]), np.isnan(b[k])), k
        assert np.array_equal(a[k][~f & ~np.isnan(a[k])], b[k][~f & ~np.isnan(a[k])]), k
        if not k.startswith("v"):
            err, scale = np.abs(a[k][f] / 4 - b[k][f] / 4).max(), np.abs(a[k][f] / 4).max()
            assert err <= (1e-11 if prec == 0 else 2e-5) * scale, (k, err, scale)
