"""Multi-shift contexts without the kept residuals (compact): the same iterates
and solutions bit for bit, the vectors they hold, and the fall-back to this form
where the others do not fit."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import helmholtz
from tests.gpu_memory import free_bytes
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

KAPS = [-1.68 - 1.66j, 0.236 - 0.926j, 2.0 + 0.5j, 40.0 + 3.0j, 400.0 - 20.0j]
GRIDS = [((12, 10, 14), (0.45, 0.4, 0.5)), ((9, 20, 30), (0.4, 0.45, 0.5))]     # bricks, march


def _both(shape, h, kaps, tol, maxit, seed):
    torch = torch_cuda()
    rng = np.random.default_rng(43)
    f = to_dev(rng.normal(size=shape) + 1j * rng.normal(size=shape))
    out = []
    for compact in (False, True):
        ms = ofd.MultiShift(shape, h, 6, max_shifts=len(kaps))
        assert not ms.compact                     # a small grid keeps the residuals
        ms.compact = compact
        assert ms.compact == compact
        xs = [torch.full(shape, complex(3.0, 1.0), dtype=torch.complex128, device="cuda") for _ in kaps]
        _, st, used = ms.solve(kaps, f, xs, tol, maxit, seed, allow_not_converged=True)
        ms.close()
        out.append((xs, [(s["iters"], s["status"], s["rel_res"]) for s in st], used))
    return f, out


@pytest.mark.parametrize("grid", GRIDS)
@pytest.mark.parametrize("seed", [0, 2])
@pytest.mark.parametrize("steps", [0, 1, 2, 3, 4, 5, 8, 9])
def test_same_iterates(grid, seed, steps):
    shape, h = grid
    announce("multishift compact", shape, seed, steps)
    torch = torch_cuda()
    _, (a, b) = _both(shape, h, KAPS, 1e-300, steps, seed)
    assert a[1:] == b[1:]
    for x, y in zip(a[0], b[0]):
        assert torch.equal(x, y)


# 1e-6: shifts freeze inside blocks; 1e-14: correction solves (true residuals
# above the tolerance); one shift: no direction beside the seed's
@pytest.mark.parametrize("kaps,tol", [(KAPS, 1e-6), (KAPS, 1e-14), (KAPS[1:2], 1e-10)])
@pytest.mark.parametrize("grid", GRIDS)
def test_same_solutions(grid, kaps, tol):
    shape, h = grid
    announce("multishift compact solves", shape, len(kaps), tol)
    torch = torch_cuda()
    f, (a, b) = _both(shape, h, kaps, tol, 10000, -1)
    assert a[1:] == b[1:]
    for x, y, kap in zip(a[0], b[0], kaps):
        assert torch.equal(x, y)
        if tol > 1e-12:
            assert helmholtz.residual(to_host(y), to_host(f), kap, h) <= 1.0001 * tol


def test_compact_where_the_rest_does_not_fit():
    """Four shifts hold 7 vectors at least and 13 with the kept residuals; 10
    are free."""
    torch = torch_cuda()
    shape, h = (320, 400, 500), (0.4, 0.4, 0.4)
    vec = 16 * 320 * 400 * 500
    announce("multishift compact by memory", shape)
    kaps = [40.0 + 3.0j, 60.0 - 5.0j, 90.0 + 1.0j, 400.0 - 20.0j]
    f = torch.ones(shape, dtype=torch.complex128, device="cuda")
    xs = [torch.empty_like(f) for _ in kaps]
    with free_bytes(10 * vec):
        ms = ofd.MultiShift(shape, h, 6, max_shifts=4)
        assert ms.compact
        with pytest.raises(ofd.OfdftError) as e:
            ms.compact = False
        assert e.value.status == ofd.NO_MEMORY and ms.compact
        status, st, _ = ms.solve(kaps, f, xs, 1e-10, 100)
        assert status == ofd.OK
    ms.compact = False                            # now they fit
    assert not ms.compact
    ms.close()
    # L_h 1 = 0: u = 1 / kappa
    for x, kap in zip(xs, kaps):
        x -= 1.0 / kap
        assert float(torch.view_as_real(x).abs().max()) <= 1e-10 * abs(1.0 / kap)
