"""Multigrid Poisson with two ring slots (compact) against the same solver with
four: iterates and solutions are the same bit for bit at step counts in and
around both rings, captured and not, for a hierarchy of two levels and of one;
the fall-back to two slots where four do not fit."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from tests.gpu_memory import free_bytes
from tests.gpu_util import announce, to_dev, torch_cuda

pytestmark = pytest.mark.gpu

H = (0.45, 0.4, 0.5)


@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("mode", [ofd.MULTIGRID, ofd.MULTIGRID_F64])
@pytest.mark.parametrize("shape", [(16, 24, 16), (12, 10, 14)])
@pytest.mark.parametrize("steps", [0, 1, 2, 3, 4, 5, 7, 8, 9, 100000])
def test_same_iterates(graphs, mode, shape, steps):
    torch = torch_cuda()
    announce("pcg compact", graphs, mode, shape, steps)
    rng = np.random.default_rng(62)
    g, x0 = to_dev(rng.normal(size=shape)), to_dev(rng.normal(size=shape))
    ps = ofd.PoissonSolver(shape, H, 6, mode)
    assert not ps.compact                         # a small grid takes four slots
    ps.set_graphs(graphs)
    out = []
    for compact in (False, True, False):          # the third: slots taken again
        ps.compact = compact
        assert ps.compact == compact
        for _ in range(2):                        # the second replays the captured block
            x = x0.clone()
            st = ps.solve(g, x, 1e-300 if steps < 100 else 1e-11, max_iter=steps, allow_not_converged=True)
            out.append((x, st["iters"], st["status"], st["rel_res"]))
    ps.close()
    assert out[0][1] == steps or (steps == 100000 and out[0][2] == ofd.OK)
    for o in out[1:]:
        assert o[1:] == out[0][1:] and torch.equal(o[0], out[0][0])


def test_other_solvers_have_no_compact_form():
    torch_cuda()
    ps = ofd.PoissonSolver((12, 10, 14), H, 6, ofd.PLAIN_F64)
    assert not ps.compact
    with pytest.raises(ofd.OfdftError) as e:
        ps.compact = True
    assert e.value.status == ofd.INVALID_ARG
    ps.close()


def test_two_slots_where_four_do_not_fit():
    """Six vectors and the levels' (FP32: 4 B per point and 12 on an eighth of
    it, and so on: 0.7 vectors) with two slots, two more with four; 8.2 are
    free."""
    torch = torch_cuda()
    shape, h = (512, 512, 512), 0.4
    vec = 8 * 512 ** 3
    announce("pcg compact by memory", shape)
    wave = torch.cos(2.0 * np.pi * torch.arange(512, dtype=torch.float64, device="cuda") / 512)
    g = wave.expand(shape).contiguous()
    x = torch.zeros_like(g)
    with free_bytes(int(8.2 * vec)):
        ps = ofd.PoissonSolver(shape, (h,) * 3, 6, ofd.MULTIGRID)
        assert ps.compact
        with pytest.raises(ofd.OfdftError) as e:
            ps.compact = False
        assert e.value.status == ofd.NO_MEMORY and ps.compact
        st = ps.solve(g, x, 1e-8)
    assert st["status"] == ofd.OK and st["rel_res"] <= 1e-8
    ps.compact = False
    assert not ps.compact
    y = torch.zeros_like(g)
    ps.solve(g, y, 1e-8)
    ps.close()
    assert torch.equal(x, y)
