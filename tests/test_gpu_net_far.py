"""The network on a volume whose planes span more than a buffer load reaches
(3400 x 3400 x 4: six planes of 16 channels at level 0, and of the parent that
the last up layer reads, are more than 2 GiB, so every convolution there takes
64-bit offsets).  Input and target are zero but in the far corner, and all
biases are zero, so there it has to give what a small volume with the same
corner gives: the output bit for bit, the gradients within the bars of
test_gpu_net.py (2e-2 of the norm; the two losses' divisors round the output
gradients differently)."""
import numpy as np
import pytest

from gpu_common import say
from test_gpu_net import net, rel, to_flat, to_list

pytestmark = pytest.mark.gpu


def test_far_corner_of_a_large_volume():
    n_large, n_small, corner, base = 3400, 64, 24, 32
    r = np.random.Generator(np.random.PCG64(12))
    xc, tc = r.standard_normal((4, corner, corner, 16)), r.standard_normal((4, corner, corner, 4)) * 0.1
    weights, got = None, {}
    for n in (n_small, n_large):
        say("far corner", n)
        g = net(n, n, 4, base=base, samples=1)
        if weights is None:
            ps = to_list(g.get_params(), base)
            ps[-1] = (r.standard_normal(ps[-1][0].shape) * 0.05, ps[-1][1])
            weights = to_flat([(w, 0.0 * b) for w, b in ps])
        g.set_params(weights)
        x, t = np.zeros(g.dims + (16,), np.float32), np.zeros(g.dims + (4,), np.float32)
        x[:, -corner:, -corner:] = xc
        t[:, -corner:, -corner:] = tc
        g.set_sample(0, x=x, t=t)
        del x, t
        y = g.forward(0)
        assert not y[:, :n - n_small].any() and not y[:, :, :n - n_small].any()
        got[n] = y[:, n - n_small:, n - n_small:].copy(), *g.gradient(0)
        say("loss", got[n][1])
        g.close()
        del g, y
    (ya, la, ga), (yb, lb, gb) = got[n_small], got[n_large]
    assert np.abs(ya).max() > 0 and np.array_equal(ya, yb)
    faces = lambda n: 2 * (n - 1) * n * 4 + n * n * 3
    scale = faces(n_large) / faces(n_small)
    assert lb * scale == pytest.approx(la, rel=1e-5)
    for l, ((wa, ba), (wb, bb)) in enumerate(zip(to_list(ga, base), to_list(gb, base))):
        for what, a, b in (("W", wa, wb), ("b", ba, bb)):
            e = rel(b * scale, a)
            say("layer", l, what, e)
            assert e < 2e-2, (l, what, e)
