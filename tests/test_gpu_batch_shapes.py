"""Every tile shape that a batch can run, forced on all its models: the same
iteration counts and the same bits as with the shapes it takes by itself, on
models of several tiles of every shape, FP64 and FP32 fields (the FP64
finishing sweeps of the latter run in the shape as well)."""
import ctypes as C

import numpy as np
import pytest

from ep_workloads import Model
from gpu_common import IT2, say

pytestmark = pytest.mark.gpu


def models():
    base = dict(ndim=2, dt=5e-4, tol=1e-6, c0=1.4e-3, freeze_iter=1200, max_iter=20000)
    return [Model(nx=160, ny=73, ly=0.5, **base), Model(nx=121, ny=64, ly=0.5, incl_radius=0.15, **base),
            Model(nx=57, ny=131, ly=1.0, **base)]


def run(prec, shape=None):
    from paper_2305_01701_amd import ep
    b = ep.Batch(models(), precision=prec)
    if shape is not None:
        use = ep.lib()._ZN2ep15batch_use_shapeEP8ep_batchi
        use.argtypes, use.restype = [C.c_void_p, C.c_int], C.c_int
        assert use(b.b, shape) == 0
    sts = [b.load_step() for _ in range(3)]
    out = [[(s["status"], s["iters"], s["iters_fp32"], s["n_yield"]) for s in st] for st in sts]
    fields = [{k: b.model(i).get(k) for k in IT2 + ["eps_p"]} for i in range(b.n)]
    b.close()
    return out, fields


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_every_shape_gives_the_same_bits(prec):
    ref, fr = run(prec)
    say("batch shapes, prec", prec, ref[-1])
    assert all(s[0] == 0 for st in ref for s in st) and all(max(st[i][3] for st in ref) > 20 for i in range(3))
    for shape in range(10):
        say("shape", shape)
        out, f = run(prec, shape)
        assert out == ref, shape
        for i in range(3):
            for k in fr[i]:
                assert np.array_equal(f[i][k], fr[i][k]), (shape, i, k)


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_checks_every_two_sweeps_equal_single_models(prec):
    """n_check = 2: launches of one sweep, on their own tiles."""
    from gpu_common import solver
    from paper_2305_01701_amd import ep
    ms = [m.with_(n_check=2, max_iter=60) for m in models()] + [Model(ndim=2, nx=700, ny=500, n_check=2, max_iter=60)]
    b = ep.Batch(ms, precision=prec)
    names = IT2 + ["p_old"]
    r = np.random.Generator(np.random.PCG64(9))
    alone = []
    for i, m in enumerate(ms):
        g = solver(m, precision=prec)
        v = g.get("vx") + 1e-3 * r.standard_normal(g.size("vx"))
        g.set("vx", v)
        b.model(i).set("vx", v)
        alone.append((g, g.load_step(), g.history()[0]))
    st = b.load_step()
    for i, (g, s, hist) in enumerate(alone):
        say("n_check 2", prec, i, st[i]["iters"], s["iters"])
        assert st[i]["iters"] == s["iters"] and np.array_equal(b.model(i).history()[0], hist)
        for k in names:
            assert np.array_equal(b.model(i).get(k), g.get(k)), (i, k)
        g.close()
    b.close()
