"""The fused 3D sweep where the planes of a chunk reach beyond 2 GiB (planes of
196 MB in FP64): the same state swept by the fused and by the unfused kernels,
update and check sweeps and the physical evaluation.  Bars as for the other
single sweeps: fields within 1e-11 of their scale, residuals within 1e-9."""
import numpy as np
import pytest
import torch

from ep_workloads import Model
from gpu_common import say

pytestmark = pytest.mark.gpu


def test_fused_sweep_of_long_planes_matches_unfused():
    from paper_2305_01701_amd import ep
    m = Model(ndim=3, nx=4959, ny=4950, nz=3, lz=0.1)
    r = np.random.Generator(np.random.PCG64(11))
    coh = np.full(m.n_cells, m.c0)
    coh[:: 7] *= 0.5
    stress = ("p", "txx", "tyy", "txy", "txz", "tyz")
    names = ("vx", "vy", "vz") + stress
    got = {}
    noise = 1e-3 * r.standard_normal(1 << 22)
    for form in (ep.EP_SWEEP_UNFUSED, ep.EP_SWEEP_FUSED):
        s = ep.Solver(m, coh, sweep=form)
        for k, n in enumerate(names):
            v = s.get(n)
            v += np.resize(np.roll(noise, 1000 * k), v.size) * (2.0 if n[0] == "v" else 1.0)
            s.set(n, v)
        say("long planes, form", form)
        res = s.residual()
        resid = s.sweep(3)
        got[form] = (res, resid, {n: s.get(n) for n in names})
        s.close()
        del s
        torch.cuda.empty_cache()
    (ra, sa, a), (rb, sb, b) = got[ep.EP_SWEEP_UNFUSED], got[ep.EP_SWEEP_FUSED]
    for k in ra:
        assert abs(ra[k] - rb[k]) <= 1e-9 * abs(ra[k]), (k, ra[k], rb[k])
    assert abs(sa - sb) <= 1e-9 * sa
    sv = max(np.abs(a[n]).max() for n in names[:3])
    ss = max(np.abs(a[n]).max() for n in stress)
    for n in names:
        e = np.abs(a[n] - b[n]).max() / (sv if n[0] == "v" else ss)
        say(n, e)
        assert e <= 1e-11, (n, e)
