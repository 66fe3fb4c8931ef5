"""Blocks of the warm-start network's kernels.  The grids choose, in the
convolutions, the blocks of 8 rows (32 and 16 output channels) and of 2 rows
with 32 channels, each with ragged blocks in x, y and z, and, in the weight
gradients, each kind of ring (rows up to 157, 328 and more voxels) and levels
down to one voxel; forward pass and gradients against the float64 oracle with
the bars of test_gpu_net.py (2e-2 of the norm, every entry of a layer's
gradient within 3e-2 of its largest)."""
import numpy as np
import pytest

from ep_workloads import Model
from gpu_common import say
from oracle import warmstart as W
from test_gpu_net import net, random_net, rel, to_list

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,base", [((70, 65, 66), 32), ((70, 65, 66), 16), ((45, 51, 46), 32),
                                       ((200, 6, 5), 32), ((341, 5, 9), 32), ((4, 4, 4), 16)],
                         ids=["8rows-32", "8rows-16", "2rows-32", "rows-200", "rows-341", "one-voxel"])
def test_forward_and_gradient_match_oracle(grid, base):
    say("net blocks", grid, base)
    n = net(*grid, base=base, samples=1)
    ps = random_net(n, base, seed=7)
    r = np.random.Generator(np.random.PCG64(8))
    x = r.standard_normal(n.dims + (16,))
    t = r.standard_normal(n.dims + (4,)) * 0.1
    n.set_sample(0, x=x, t=t)
    y = n.forward(0)
    yr, cache = W.forward(ps, x, store=W.bf16)
    assert rel(y, yr) < 2e-2
    assert np.abs(y - yr).max() < 5e-2 * np.abs(yr).max()
    nx, ny, nz = grid
    zero = {k: np.zeros((nx + (k == "vx")) * (ny + (k == "vy")) * (nz + (k == "vz"))) for k in ("vx", "vy", "vz")}
    _, mask = W.targets(Model(ndim=3, nx=nx, ny=ny, nz=nz), zero, 1.0)
    t16 = np.zeros(n.dims + (16,))
    t16[..., :3] = t[..., :3].astype(np.float32)
    _, gy = W.loss_grad(yr, t16, mask)
    gr = W.backward(cache, gy, store=W.bf16)
    gl = to_list(n.gradient(0)[1], base)
    for l in range(W.N_LAYERS):
        for q, what in enumerate("Wb"):
            e = rel(gl[l][q], gr[l][q])
            m = float(np.abs(gl[l][q] - gr[l][q]).max() / np.abs(gr[l][q]).max())
            say("layer", l, "d" + what, e, m)
            assert e < 2e-2 and m < 3e-2, (l, what, e, m)
    n.close()
