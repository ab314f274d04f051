"""When the network-preconditioned flexible CG gives way to plain CG after its
first look (10x in 20 iterations): not while it converges, however unevenly, and
once it stalls (less than 2x in 200 iterations).  The networks are set by hand:
their outputs are known functions of the residual."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import nn, poisson
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

CENTRE, XM, XP = 13, 12, 14
H = (0.4, 0.4, 0.4)


def _network(out):
    """Channels 0 and 1 carry max(r, 0) and max(-r, 0) from the input to the last
    layer, `out` maps taps to their two weights there."""
    w = {name: np.zeros((27, ci, co)) for name, ci, co in nn.LAYERS}
    w["c0a"][CENTRE, 0, :2] = 1.0, -1.0
    for name, first in (("c0b", 0), ("d0a", 32), ("d0b", 0)):      # the skip channels follow 32 upsampled ones
        for k in range(2):
            w[name][CENTRE, first + k, k] = 1.0
    for tap, pair in out.items():
        w["out"][tap, :2, 0] = pair
    net = ofd.Network(0)
    net.set_precision(True)
    net.set_weights(w)
    return net


def _solve(net, g, tol):
    s = ofd.PoissonSolver(g.shape, H, 6, ofd.LEARNED)
    s.set_network(net)
    s.set_learned_mode(True)
    x = to_dev(np.zeros(g.shape))
    st = s.solve(to_dev(g), x, tol)
    s.close()
    assert st["status"] == ofd.OK and poisson.residual(to_host(x), g, H) <= tol
    return st


def test_uneven_convergence_goes_on():
    """z = r where r > 0, 0.05 r elsewhere: 14x in the first 20 iterations (of the
    high-frequency part), then 4 to 5x in 20 and 200 to the tolerance."""
    torch_cuda()
    announce("learned uneven")
    n = 24
    alt = (-1.0) ** np.arange(n)
    g = alt[:, None, None] * alt[:, None] * alt + 0.03 * np.random.default_rng(1).normal(size=(n, n, n))
    g -= g.mean()
    st = _solve(_network({CENTRE: (1.0, -0.05)}), g, 1e-8)
    assert st["fell_back"] == 0 and 100 < st["iters"] < 400


def test_stalled_run_is_given_up():
    """z = -d^2 r / dx^2 but for 1e-5 max(r, 0): the part of g that varies in x is
    gone after 20 iterations, the rest hardly moves."""
    torch_cuda()
    announce("learned stall")
    n = 16
    rng = np.random.default_rng(2)
    xp, yz = rng.normal(size=n), rng.normal(size=(n, n))
    g = (xp - xp.mean()) + 0.01 * (yz - yz.mean())[:, :, None]
    st = _solve(_network({CENTRE: (2.0 + 1e-5, -2.0), XM: (-1.0, 1.0), XP: (-1.0, 1.0)}), g, 1e-8)
    # one application for the start, one for z_0 and one per iteration to the look that ends it
    assert st["fell_back"] == 1 and st["nn_applies"] in (221, 421)
