"""Field transfers on both sides of the size up to which a field is copied with
its padding and unpacked on the host: what was set comes back, the fields
around it stay, and the derived stress is that of the two it is derived from."""
import numpy as np
import pytest

from ep_workloads import Model
from gpu_common import it_names, say, solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid", [(8, 3), (63, 63), (191, 206), (191, 208), (383, 191), (5, 4, 3), (31, 31, 31), (31, 34, 36),
                                  (63, 23, 25), (95, 60, 40)], ids=lambda g: "x".join(map(str, g)))
def test_fields_set_and_read_back(grid):
    m = Model(ndim=len(grid), nx=grid[0], ny=grid[1], nz=grid[2] if len(grid) == 3 else 1)
    say("fields", grid)
    g = solver(m)
    r = np.random.Generator(np.random.PCG64(4))
    names = [n for n in it_names(m) if n != "tzz"] + ["p_old", "ux", "exx", "eps_p", "cohesion"]
    put = {n: r.standard_normal(g.size(n)) for n in names}
    for n in names:
        g.set(n, put[n])
    for _ in range(2):
        for n in names:
            assert np.array_equal(g.get(n), put[n]), n
        if m.ndim == 3:
            assert np.array_equal(g.get("tzz"), -(put["txx"] + put["tyy"]))
    g.close()
