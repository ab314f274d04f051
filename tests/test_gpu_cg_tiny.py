"""Poisson CG of grids that fit one workgroup (every iteration in one launch):
axes at the smallest size, short last plane groups, the largest grid of each
planes-per-thread choice and one just past it, against the oracle's CG iterates
at fixed step counts and against the residual at convergence; the outcomes of
the iteration cap, a zero and a non-finite right-hand side."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import poisson
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

SHAPES = [(6, 6, 6), (6, 7, 40), (9, 13, 6), (16, 16, 16), (20, 20, 20), (31, 8, 32), (8, 32, 32), (21, 20, 20)]
H = (0.4, 0.45, 0.5)


def _solve(shape, g, tol, maxit, mode):
    s = ofd.PoissonSolver(shape, H, 6, mode)
    phi = to_dev(np.zeros(shape))
    st = s.solve(to_dev(g), phi, tol, maxit, allow_not_converged=True)
    s.close()
    return to_host(phi), st


@pytest.mark.parametrize("steps", [1, 2, 7])
@pytest.mark.parametrize("shape", SHAPES)
def test_iterates(shape, steps):
    torch_cuda()
    announce("tiny cg", shape, steps)
    g = np.random.default_rng(sum(shape)).normal(size=shape)
    x, st = _solve(shape, g, 1e-14, steps, ofd.PLAIN_F64)
    ref, it, _ = poisson.solve_cg(g - g.mean(), H, tol=1e-300, maxit=steps)
    assert st["iters"] == steps == it and st["status"] == ofd.NOT_CONVERGED
    ref = ref - ref.mean()
    assert np.abs(x - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("mode,tol", [(ofd.PLAIN_F64, 1e-11), (ofd.REFINED_F32, 1e-10)])
@pytest.mark.parametrize("shape", SHAPES)
def test_converged(shape, mode, tol):
    torch_cuda()
    announce("tiny cg converged", shape, mode)
    g = np.random.default_rng(sum(shape)).normal(size=shape)
    x, st = _solve(shape, g, tol, 100000, mode)
    assert st["status"] == ofd.OK and poisson.residual(x, g - g.mean(), H) <= tol


def test_outcomes():
    torch_cuda()
    shape = (16, 16, 16)
    x, st = _solve(shape, np.ones(shape), 1e-10, 100, ofd.PLAIN_F64)
    assert st["iters"] == 0 and np.abs(x).max() == 0.0
    g = np.random.default_rng(0).normal(size=shape)
    g[3, 4, 5] = np.nan
    s = ofd.PoissonSolver(shape, H, 6)
    with pytest.raises(ofd.OfdftError) as e:
        s.solve(to_dev(g), to_dev(np.zeros(shape)), 1e-10)
    assert e.value.status == ofd.NONFINITE
    s.close()
