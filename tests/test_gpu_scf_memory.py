"""A fixed-point context created with too little free memory for its solvers'
optional vectors does without them: it is created all the same, and its state
and first step are the same bit for bit."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from tests.gpu_memory import free_bytes
from tests.gpu_util import announce, torch_cuda

pytestmark = pytest.mark.gpu


def _setup(n, h, tol, history, mg, dtype=ofd.C128):
    """run(step) creates a context on an n^3 grid, takes a step if wanted and
    returns the free bytes after creation and the state vectors."""
    torch = torch_cuda()
    ax = 2.0 * np.pi * torch.arange(n, dtype=torch.float64, device="cuda") / n
    rho = 0.03 * (1.0 + 0.2 * torch.cos(ax)[:, None, None] + 0.1 * torch.sin(ax)[:, None] + 0.05 * torch.cos(ax))
    rho = rho.expand(n, n, n).contiguous()
    b = -rho * (1.0 + 0.1 * torch.cos(ax))
    b -= b.mean() + rho.mean()
    electrons = float(rho.sum()) * h ** 3
    u0 = rho.sqrt()
    kw = dict(lam=0.2, mu=1, history=history, zeta=0.3, u_tol=1e-6, poisson_tol=tol, helmholtz_tol=tol,
              poisson_mode=ofd.MULTIGRID if mg else ofd.PLAIN_F64,
              helmholtz_dtype=dtype,
              helmholtz_precond=ofd.PRECOND_MULTIGRID if mg and dtype == ofd.C128 else ofd.PRECOND_NONE,
              u_precond=ofd.PRECOND_MULTIGRID if mg else ofd.PRECOND_NONE, helmholtz_multishift=not mg)

    def run(step):
        ctx = ofd.SCF((n,) * 3, (h,) * 3, b, u0, electrons, **kw)
        left = torch.cuda.mem_get_info()[0]
        if step:
            ctx.step()
        out = [ctx.get(k, rho).cpu() for k in (ofd.SCF.V, ofd.SCF.U, ofd.SCF.PHI, ofd.SCF.VLR)]
        ctx.close()
        return left, out

    return run


# Optional, in real vectors: two complex ones of each of the four systems, two of
# the multigrid Poisson solver: 18, of which half are missing.  With the
# multi-shift start 16, and while its context lives 10 to 22 more than afterwards:
# 8 more are there.
@pytest.mark.parametrize("mg,missing", [(True, 9), (False, -8)])
def test_context_without_room(mg, missing):
    torch = torch_cuda()
    n = 320
    announce("scf memory", n, mg)
    run = _setup(n, 0.45, 1e-6, 3, mg)
    run(True)                                     # what the runtime keeps from a first run
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    left, full = run(True)
    with free_bytes(before - left - missing * 8 * n ** 3):
        _, short = run(True)
    for x, y in zip(full, short):
        assert torch.equal(x, y)


def test_later_parts_lack_the_room():
    """In real vectors: the complex64 batch takes its 8 optional ones where 18 (a
    sixteenth of the card at this size) stay free, and the Poisson solver (7) and
    the mixing history (18) allocated after it then do not fit.  10 optional ones
    in all, of which 5 are missing."""
    torch = torch_cuda()
    n = 512
    announce("scf memory, second attempt", n)
    run = _setup(n, 0.45, 1e-3, 8, True, ofd.C64)
    run(False)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    left, full = run(False)
    with free_bytes(before - left - 5 * 8 * n ** 3):
        _, short = run(False)
    assert "anderson" in ofd.last_error()         # where the first attempt stopped
    for x, y in zip(full, short):
        assert torch.equal(x, y)
