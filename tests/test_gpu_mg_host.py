"""A multigrid cycle's launches cost the host no more on a large grid than on a
small one: what a launch needs of the grid alone is found at creation."""
import time

import pytest

import paper_1412_8250_amd as ofd
from tests.gpu_util import announce, torch_cuda

pytestmark = pytest.mark.gpu


def _enqueue_time(n):
    """Host seconds of one cycle of an n^3 grid, the device's time aside (best of
    many short runs that the queue takes in whole)."""
    torch = torch_cuda()
    r = torch.ones((n, n, n), dtype=torch.float64, device="cuda")
    z = torch.empty_like(r)
    ps = ofd.PoissonSolver((n, n, n), (0.4,) * 3, 6, ofd.MULTIGRID)
    best = float("inf")
    for _ in range(30):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(4):
            ps.apply_preconditioner(r, z)
        best = min(best, (time.perf_counter() - t) / 4)
    torch.cuda.synchronize()
    ps.close()
    return best


def test_large_grids_take_no_more_host_time():
    # 64^3: three levels; 512^3: six, so 11 launches in place of 5, and a tenth for noise
    small, large = _enqueue_time(64), _enqueue_time(512)
    announce("cycle host time", small, large)
    assert large <= 2.4 * small
