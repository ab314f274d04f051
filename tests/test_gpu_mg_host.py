"""A multigrid cycle's launches cost the host no more on a large grid than on a
small one (what a launch needs of the grid alone is found at creation), and its
hierarchy holds no array that no kernel uses."""
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


@pytest.mark.parametrize("kind,elem", [(ofd.PRECOND_MULTIGRID, 8), (ofd.PRECOND_MULTIGRID_F64, 16)])
def test_hierarchy_holds_what_it_uses(kind, elem):
    """z; u on the finest level; u, f and t on the levels below (256^3 has 4 of
    them: 1/8 + 1/64 + 1/512 + 1/4096 of the points)."""
    torch = torch_cuda()
    n = 256
    announce("hierarchy memory", kind)
    b = ofd.HelmholtzBatch([(n,) * 3], [(0.4,) * 3])
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    b.set_preconditioner(kind)
    used = before - torch.cuda.mem_get_info()[0]
    b.close()
    coarse = 1 / 8 + 1 / 64 + 1 / 512 + 1 / 4096
    # each allocation is a whole number of 2 MiB pages; streams and events besides
    assert used <= n ** 3 * (16 + elem * (1 + 3 * coarse)) + (64 << 20)
