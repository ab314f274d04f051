"""Multigrid Poisson: the ring of preconditioned residuals from which p and x
are brought up to date, at iteration counts in and around it, captured and
not, against flexible CG iterates formed by the oracle's operators; the two
ring lengths give the same iterates."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import fd, multigrid
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

SHAPE, H = (16, 24, 16), (0.45, 0.4, 0.5)


def _fcg(g, x, steps):
    x = x.copy()
    g = g - g.mean()
    r = g + fd.laplacian(x, H, 6)
    z = multigrid.vcycle(r, H)
    p = z
    rz = (r * z).sum()
    for _ in range(steps):
        q = -fd.laplacian(p, H, 6)
        alpha = rz / (p * q).sum()
        x += alpha * p
        old, r = r, r - alpha * q
        z = multigrid.vcycle(r, H)
        beta = (z * (r - old)).sum() / rz
        rz = (r * z).sum()
        p = z + beta * p
    return x - x.mean()


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 7, 8, 9])
def test_iterates_around_the_ring(graphs, steps):
    torch_cuda()
    announce("pcg ring", graphs, steps)
    rng = np.random.default_rng(61)
    g, x0 = rng.normal(size=SHAPE), rng.normal(size=SHAPE)
    ps = ofd.PoissonSolver(SHAPE, H, 6, ofd.MULTIGRID_F64)
    ps.set_graphs(graphs)
    x = to_dev(x0)
    st = ps.solve(to_dev(g), x, 1e-300, max_iter=steps, allow_not_converged=True)
    ps.close()
    assert st["iters"] == steps
    ref = _fcg(g, x0, steps)
    # up to 9 recurrence steps of rounding, and the FP64 cycle matches its
    # reference to 1e-12 in each of them; |x0 - x| is of the size of x
    assert np.abs(to_host(x) - ref).max() <= 1e-10 * np.abs(x0).max()


def test_two_slots_on_a_large_grid():
    """Eight vectors of this grid are more than an eighth of the card's memory
    (288 GB), so the solver keeps two slots.  A plane wave of the smallest
    eigenvalue: the relative error of phi is at most the relative residual."""
    torch = torch_cuda()
    shape, h = (768, 896, 896), (0.4, 0.4, 0.4)
    announce("pcg ring of two", shape)
    wave = torch.cos(2.0 * np.pi * torch.arange(shape[2], dtype=torch.float64, device="cuda") / shape[2])
    lam = -float(fd.symbol_1d(shape[2], h[0], 6)[1])
    g = wave.expand(shape).contiguous()
    x = torch.zeros_like(g)
    ps = ofd.PoissonSolver(shape, h, 6, ofd.MULTIGRID)
    st = ps.solve(g, x, 1e-8)
    ps.close()
    assert 1 <= st["iters"] <= 30 and st["rel_res"] <= 1e-8
    x -= g / abs(lam)
    # |x - g / lam| <= |residual| / lam, and rounding of the stencil (1e-15 of
    # the weights' size against lam: 1e-15 * 71 / lam)
    bound = (1e-8 + 1e-13 / abs(lam)) / abs(lam)
    assert float(torch.linalg.vector_norm(x)) <= bound * float(torch.linalg.vector_norm(g))
