"""Products of z formed in the cycle's last kernel (and, on grids that are
their own coarsest level, by a pass of their own): iterates of the
preconditioned loops after a few steps against the oracle's, on a one-level
grid, on several tiles and z chunks, and in batches whose groups mix both; the
FP32 cycle converges as the FP64 one does."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import fd, helmholtz, multigrid
from tests.gpu_util import announce, to_dev, to_host, torch_cuda
from tests.test_gpu_batch_ring import KAPS, _cocg, _solve

pytestmark = pytest.mark.gpu

ONE, TWO, MANY = (14, 10, 12), (16, 24, 16), (64, 48, 96)
H = (0.45, 0.4, 0.5)
STEPS = 3


@pytest.mark.parametrize("shapes", [(ONE,), (MANY,), (TWO, TWO, TWO), (TWO, ONE, ONE, MANY), (MANY, MANY, ONE)])
def test_cocg_iterates(shapes):
    torch_cuda()
    announce("mg products cocg", shapes)
    rng = np.random.default_rng(71)
    n = len(shapes)
    kaps = [KAPS[j % 3] for j in range(n)]
    f = [rng.normal(size=s) + 1j * rng.normal(size=s) for s in shapes]
    x0 = [rng.normal(size=s) + 1j * rng.normal(size=s) for s in shapes]
    xs = [to_dev(x) for x in x0]
    _solve(list(shapes), [H] * n, kaps, [to_dev(v) for v in f], xs, STEPS, True)
    for j in range(n):
        ref = _cocg(f[j], x0[j], kaps[j], H, STEPS, True)
        # the FP64 cycle matches its reference to 1e-12 in each step
        assert np.abs(to_host(xs[j]) - ref).max() <= 3e-11 * np.abs(ref).max()


@pytest.mark.parametrize("shape", [ONE, MANY])
def test_poisson_iterates(shape):
    torch_cuda()
    announce("mg products poisson", shape)
    rng = np.random.default_rng(72)
    g, x0 = rng.normal(size=shape), rng.normal(size=shape)
    ps = ofd.PoissonSolver(shape, H, 6, ofd.MULTIGRID_F64)
    xd = to_dev(x0)
    ps.solve(to_dev(g), xd, 1e-300, max_iter=STEPS, allow_not_converged=True)
    ps.close()
    x, r = x0.copy(), g - g.mean() + fd.laplacian(x0, H, 6)
    p = z = multigrid.vcycle(r, H)
    rz = (r * z).sum()
    for _ in range(STEPS):
        q = -fd.laplacian(p, H, 6)
        alpha = rz / (p * q).sum()
        x += alpha * p
        r = r - alpha * q
        z = multigrid.vcycle(r, H)
        beta = -alpha * (z * q).sum() / rz
        rz = (r * z).sum()
        p = z + beta * p
    assert np.abs(to_host(xd) - (x - x.mean())).max() <= 3e-11 * np.abs(x0).max()


def test_fp32_cycle_takes_the_same_steps():
    torch = torch_cuda()
    announce("mg products fp32")
    rng = np.random.default_rng(73)
    f = to_dev(rng.normal(size=MANY) + 1j * rng.normal(size=MANY))
    its = {}
    for kind in (ofd.PRECOND_MULTIGRID, ofd.PRECOND_MULTIGRID_F64):
        b = ofd.HelmholtzBatch([MANY] * 2, [H] * 2, 6, ofd.C128)
        b.set_preconditioner(kind)
        xs = [torch.zeros_like(f) for _ in range(2)]
        _, st = b.solve(KAPS[:2], [f, f], xs, 1e-8)
        b.close()
        its[kind] = [s["iters"] for s in st]
        for x, k in zip(xs, KAPS):
            assert helmholtz.residual(to_host(x), to_host(f), k, H) <= 1e-8
    # single-precision rounding of M moves a residual by 1e-6 of itself: one
    # step more or less at most
    assert all(abs(a - b) <= 1 for a, b in zip(*its.values()))
