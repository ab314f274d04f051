"""The stepped schedule's ring of directions (iterates brought up to date
every two or four iterations): step counts at and around its length, on bricks
and on the march, with and without the preconditioner, against COCG iterates
formed by the oracle's operators; a batch too large for four slots gives the
same iterates."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import helmholtz, multigrid
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

KAPS = [-1.68 - 1.66j, 0.236 - 0.926j, 2.0 + 0.5j]


def _cocg(f, x, kappa, h, steps, precond):
    x = x.copy()
    r = f - helmholtz.apply(x, kappa, h)
    p, rho = None, None
    for _ in range(steps):
        z = multigrid.vcycle(r, h, kappa) if precond else r
        rho_new = (r * z).sum()
        p = z if p is None else z + rho_new / rho * p
        rho = rho_new
        q = helmholtz.apply(p, kappa, h)
        alpha = rho / (p * q).sum()
        x += alpha * p
        r = r - alpha * q
    return x


def _solve(shapes, hs, kaps, fs, xs, steps, precond, config=None):
    b = ofd.HelmholtzBatch(shapes, hs, 6, ofd.C128)
    if config is not None:
        b.set_config(*config)
    if precond:
        b.set_preconditioner(ofd.PRECOND_MULTIGRID_F64)
    _, st = b.solve(kaps, fs, xs, 1e-300, max_iter=steps, allow_not_converged=True)
    b.close()
    return st


# default (bricks) and a marched tile shape
@pytest.mark.parametrize("config", [None, (2, 0)])
@pytest.mark.parametrize("precond", [False, True])
@pytest.mark.parametrize("steps", [0, 1, 2, 3, 4, 5, 7, 8, 9])
def test_iterates_around_the_ring(config, precond, steps):
    torch_cuda()
    announce("batch ring", config, precond, steps)
    shape, h = ((16, 24, 16), (0.45, 0.4, 0.5)) if precond else ((12, 10, 14), (0.45, 0.4, 0.5))
    rng = np.random.default_rng(51)
    f = [rng.normal(size=shape) + 1j * rng.normal(size=shape) for _ in KAPS]
    x0 = [rng.normal(size=shape) + 1j * rng.normal(size=shape) for _ in KAPS]
    xs = [to_dev(x) for x in x0]
    st = _solve([shape] * 3, [h] * 3, KAPS, [to_dev(v) for v in f], xs, steps, precond, config)
    for j, kap in enumerate(KAPS):
        assert st[j]["iters"] == steps
        ref = _cocg(f[j], x0[j], kap, h, steps, precond)
        # up to 9 recurrence steps of rounding; the FP64 cycle matches its
        # reference to 1e-12 in each of them
        tol = 1e-10 if precond else 1e-11
        assert np.abs(to_host(xs[j]) - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.parametrize("steps", [1, 4, 7])
def test_two_slots_give_the_same_iterates(steps):
    """Six vectors of the second system are more than an eighth of the card's
    memory (288 GB), so this batch keeps two slots."""
    torch = torch_cuda()
    announce("batch ring of two", steps)
    shape, h, big = (16, 24, 16), (0.45, 0.4, 0.5), (768, 704, 704)
    rng = np.random.default_rng(52)
    f = to_dev(rng.normal(size=shape) + 1j * rng.normal(size=shape))
    four, two = torch.zeros_like(f), torch.zeros_like(f)
    _solve([shape], [h], KAPS[:1], [f], [four], steps, False)
    zero = torch.zeros(big, dtype=torch.complex128, device="cuda")
    rest = torch.zeros_like(zero)
    _solve([shape, big], [h, h], KAPS[:2], [f, zero], [two, rest], steps, False)
    assert torch.equal(four, two)
    assert not bool(torch.view_as_real(rest).any())
