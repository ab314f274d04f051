"""Poisson CG of grids that fit one workgroup, over more iterations than one
launch runs: the iteration goes on where it stopped (a new start from the
iterate would take 8% and 57% more steps here), and a solve whose tolerance cannot be
met is made of bounded launches."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import poisson
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

PER_LAUNCH = 512


def _solve(shape, h, g, tol, maxit, noalloc=False):
    x = to_dev(np.zeros(shape))
    ofd.profile_reset()
    if noalloc:
        st = ofd.poisson_solve_noalloc(to_dev(g), x, h, tol, maxit, allow_not_converged=True)
    else:
        s = ofd.PoissonSolver(shape, h)
        st = s.solve(to_dev(g), x, tol, maxit, allow_not_converged=True)
        s.close()
    return to_host(x), st, ofd.profile_read()["cg_stencil"]["launches"]


@pytest.mark.parametrize("noalloc", [False, True])
# four planes a thread and eight
@pytest.mark.parametrize("shape,h", [((16, 16, 16), (1.5, 0.7, 0.02)), ((32, 8, 32), (0.05, 0.4, 2.0))])
def test_goes_on_in_the_next_launch(shape, h, noalloc):
    torch_cuda()
    announce("tiny cg launches", shape, noalloc)
    g = np.random.default_rng(5).normal(size=shape)
    g -= g.mean()
    _, want, _ = poisson.solve_cg(g, h, tol=1e-9, maxit=20000)
    assert want > PER_LAUNCH
    x, st, launches = _solve(shape, h, g, 1e-9, 20000, noalloc)
    assert st["status"] == ofd.OK and poisson.residual(x, g, h) <= 1e-9
    # rounding may shift the last steps of an ill-conditioned run
    assert abs(st["iters"] - want) <= 0.05 * want
    assert launches == -(-st["iters"] // PER_LAUNCH)


@pytest.mark.parametrize("steps", [511, 512, 513, 1024, 1025])
def test_cap_around_launches(steps):
    """Capped runs with a tolerance out of reach."""
    torch_cuda()
    announce("tiny cg cap", steps)
    shape, h = (16, 16, 16), (1.5, 0.7, 0.02)
    g = np.random.default_rng(5).normal(size=shape)
    x, st, launches = _solve(shape, h, g - g.mean(), 1e-300, steps)
    assert st["iters"] == steps and st["status"] == ofd.NOT_CONVERGED and np.isfinite(x).all()
    assert launches == -(-steps // PER_LAUNCH)


@pytest.mark.parametrize("shape,one", [((14, 20, 20), True), ((8, 32, 32), True), ((24, 16, 16), False)])
def test_which_grids_take_one_launch(shape, one):
    """Over 6000 points FP64 iterations run two launches each where every axis
    admits bricks (at least ten points)."""
    torch_cuda()
    announce("tiny cg rule", shape)
    g = np.random.default_rng(6).normal(size=shape)
    h = (0.4, 0.45, 0.5)
    x, st, launches = _solve(shape, h, g, 1e-10, 1000)
    assert st["status"] == ofd.OK and poisson.residual(x, g - g.mean(), h) <= 1e-10
    assert (launches == 1) == one
