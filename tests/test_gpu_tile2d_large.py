"""The two tile shapes that only large or long single 2D models choose (56 x 8
cells in FP32, 24 x 24 with 256 threads in FP64) against the oracle; bars as in
test_gpu_tile2d.py.  With a per-cell G a cell of the FP32 grid lies at its bound
within FP32 rounding (the unfused FP32 kernels let it yield as well, FP64 ones
and the oracle do not): there the window of sweeps has to give the bits of
single sweeps, which run on other tiles, and as many cells as such a flip
reaches in five sweeps may be off the oracle."""
import ctypes as C

import numpy as np
import pytest

from gpu_common import compare, it_names, say
from test_gpu_tile2d import pair
from test_launch_plans import lib  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_g", [False, True], ids=["uniform", "G"])
@pytest.mark.parametrize("grid,prec,shape", [((260, 1200), 1, 1), ((1601, 1600), 0, 2)], ids=["fp32", "fp64"])
def test_shapes_of_large_models(lib, grid, prec, shape, with_g):  # noqa: F811
    choice = lib._ZN2ep13tile2d_choiceEbiii
    choice.restype = C.c_int
    assert choice(C.c_bool(prec == 1), *grid, 256) == shape
    say("large 2d tiles", grid, "prec", prec, with_g)
    m, g, o = pair(grid, with_g, prec)
    names = it_names(m)
    for n in (3, 2):
        rg = g.sweep(n)
        for _ in range(n):
            ro = o.sweep()
        if prec == 1 and with_g:
            continue
        compare(m, g.fields(names), o.fields(names), names, 1e-11 if prec == 0 else 2e-5, f"{grid} {n}")
        assert abs(rg - ro) <= (1e-9 if prec == 0 else 1e-3) * ro, (n, rg, ro)
    if prec == 1 and with_g:
        _, b, _ = pair(grid, with_g, prec)
        for _ in range(5):
            b.sweep(1)
        for k in names:
            assert np.array_equal(g.get(k), b.get(k)), k
            e = np.abs(g.get(k) - o.get(k)) / np.abs(o.get(k)).max()
            assert (e > 2e-5).sum() <= 21 * 21, (k, (e > 2e-5).sum())      # 2 points a sweep on each side
        b.close()
    g.close()
    o.close()
