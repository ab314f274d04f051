"""Multi-shift COCG's deferred iterate updates: step counts at and around the
block of iterations brought up to date together, on a grid that runs bricks and
on one with a short axis that runs the march, against the oracle's iterates
element by element; shifts that freeze inside a block keep the iterate of their
own step."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import helmholtz, multishift
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

KAPS = [-1.68 - 1.66j, 0.236 - 0.926j, 2.0 + 0.5j, 40.0 + 3.0j, 400.0 - 20.0j]
GRIDS = [((12, 10, 14), (0.45, 0.4, 0.5)), ((9, 20, 30), (0.4, 0.45, 0.5))]


def _run(shape, h, f, tol, maxit):
    torch = torch_cuda()
    ms = ofd.MultiShift(shape, h, 6, max_shifts=len(KAPS))
    xs = [torch.full(shape, complex(3.0, 1.0), dtype=torch.complex128, device="cuda") for _ in KAPS]
    _, st, _ = ms.solve(KAPS, to_dev(f), xs, tol, maxit, 0, allow_not_converged=True)
    ms.close()
    return [to_host(x) for x in xs], st


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("steps", [2, 3, 5, 7, 8, 9])
def test_iterates_around_blocks(grid, steps):
    shape, h = grid
    announce("multishift block", shape, steps)
    rng = np.random.default_rng(41)
    f = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    xs, st = _run(shape, h, f, 1e-300, steps)
    ref, _, k = multishift.solve(f, KAPS, h, seed=0, tol=0.0, maxit=steps)
    assert k == steps
    for x, r, s in zip(xs, ref, st):
        assert s["iters"] == steps
        # 7 to 9 recurrence steps of rounding, as for the other fixed-step checks
        assert np.abs(x - r).max() <= 1e-11 * np.abs(r).max()


@pytest.mark.parametrize("grid", GRIDS)
def test_shifts_that_freeze_early(grid):
    shape, h = grid
    announce("multishift freeze", shape)
    rng = np.random.default_rng(42)
    f = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    xs, st = _run(shape, h, f, 1e-6, 10000)
    its = [s["iters"] for s in st]
    assert its[4] < its[3] < its[0]            # large shifts freeze long before the seed
    for x, kap, s in zip(xs, KAPS, st):
        assert helmholtz.residual(x, f, kap, h) <= 1.0001e-6
