"""Batches with two ring slots (compact) against the same batch with four: the
iterates and solutions are the same bit for bit at step counts in and around
both rings, on bricks and on the march, with and without the preconditioner, in
complex64 and in the timed schedule; the fall-back to two slots where four do
not fit, at creation and when the preconditioner's arrays need the room."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from tests.gpu_memory import free_bytes
from tests.gpu_util import announce, to_dev, torch_cuda

pytestmark = pytest.mark.gpu

KAPS = [-1.68 - 1.66j, 0.236 - 0.926j, 2.0 + 0.5j]
H = (0.45, 0.4, 0.5)


def _both(shapes, precond, dtype, config, tol, steps, timed=()):
    torch = torch_cuda()
    rng = np.random.default_rng(53)
    f = [to_dev(rng.normal(size=s) + 1j * rng.normal(size=s)) for s in shapes]
    x0 = [to_dev(rng.normal(size=s) + 1j * rng.normal(size=s)) for s in shapes]
    out = []
    b = ofd.HelmholtzBatch(shapes, [H] * len(shapes), 6, dtype)
    assert not b.compact                          # small grids take four slots
    if config is not None:
        b.set_config(*config)
    b.set_preconditioner(precond)
    ofd.profile_reset(timed)
    try:
        for compact in (False, True, False):      # the third: slots taken again
            b.compact = compact
            assert b.compact == compact
            xs = [x.clone() for x in x0]
            _, st = b.solve(KAPS[:len(shapes)], f, xs, tol, max_iter=steps, allow_not_converged=True)
            out.append((xs, [(s["iters"], s["status"], s["rel_res"]) for s in st]))
    finally:
        ofd.profile_reset()
    b.close()
    for xs, st in out[1:]:
        assert st == out[0][1]
        for x, y in zip(xs, out[0][0]):
            assert torch.equal(x, y)
    return out[0][1]


# default (bricks; the second grid has a short axis and runs the march) and a marched shape
@pytest.mark.parametrize("config", [None, (2, 0)])
@pytest.mark.parametrize("precond", [ofd.PRECOND_NONE, ofd.PRECOND_MULTIGRID, ofd.PRECOND_MULTIGRID_F64])
@pytest.mark.parametrize("steps", [0, 1, 2, 3, 4, 5, 7, 8, 9])
def test_same_iterates(config, precond, steps):
    announce("batch compact", config, precond, steps)
    # with a preconditioner: a two-level and a one-level hierarchy
    shapes = [(16, 24, 16), (12, 8, 14)] if precond else [(12, 10, 14), (9, 20, 30)]
    st = _both(shapes, precond, ofd.C128, config, 1e-300, steps)
    assert [s[0] for s in st] == [steps] * 2


@pytest.mark.parametrize("config", [None, (2, 0)])
@pytest.mark.parametrize("steps", [1, 3, 6, 100000])
def test_same_iterates_complex64(config, steps):
    announce("batch compact c64", config, steps)
    st = _both([(12, 10, 14), (9, 20, 30)], ofd.PRECOND_NONE, ofd.C64, config, 1e-10, steps)
    assert steps < 100000 or all(s[1] == ofd.OK for s in st)


# systems that stop in different iterations; every launch on its own (timed) and captured
@pytest.mark.parametrize("timed", [(), ofd.KERNEL_CLASSES])
@pytest.mark.parametrize("precond", [ofd.PRECOND_NONE, ofd.PRECOND_MULTIGRID])
def test_same_solutions(precond, timed):
    announce("batch compact solves", precond, timed)
    shapes = [(16, 24, 16), (24, 16, 32), (16, 24, 16)]
    st = _both(shapes, precond, ofd.C128, None, 1e-10, 100000, timed)
    assert all(s[1] == ofd.OK for s in st)


def test_two_slots_where_four_do_not_fit():
    """A system holds 4 vectors at least and 6 with four slots; 5 are free."""
    torch = torch_cuda()
    shape, vec = (512, 512, 512), 16 * 512 ** 3
    announce("batch compact by memory", shape)
    f = torch.ones(shape, dtype=torch.complex128, device="cuda")
    x = torch.zeros_like(f)
    with free_bytes(5 * vec):
        b = ofd.HelmholtzBatch([shape], [(0.4,) * 3])
        assert b.compact
        with pytest.raises(ofd.OfdftError) as e:
            b.compact = False
        assert e.value.status == ofd.NO_MEMORY and b.compact
        assert b.solve([40.0 + 3.0j], [f], [x], 1e-10, 100)[0] == ofd.OK
    b.compact = False
    assert not b.compact
    b.close()
    x -= 1.0 / (40.0 + 3.0j)                      # L_h 1 = 0: u = 1 / kappa
    assert float(torch.view_as_real(x).abs().max()) <= 1e-10 / 40.0


def test_preconditioner_takes_the_room_of_two_slots():
    """The batch holds 6 vectors with four slots and 4 with two, z and the levels
    (complex64: 8 B per point and 24 on an eighth of it, and so on) 1.7 more:
    with 7.2 free the preconditioner fits only beside two slots."""
    torch = torch_cuda()
    shape, vec = (512, 512, 512), 16 * 512 ** 3
    announce("batch preconditioner by memory", shape)
    f = torch.ones(shape, dtype=torch.complex128, device="cuda")
    x = torch.zeros_like(f)
    with free_bytes(int(7.2 * vec)):
        b = ofd.HelmholtzBatch([shape], [(0.4,) * 3])
        b.compact = False
        assert not b.compact
        b.set_preconditioner(ofd.PRECOND_MULTIGRID)
        assert b.compact
        assert b.solve([40.0 + 3.0j], [f], [x], 1e-10, 100)[0] == ofd.OK
    b.close()
    x -= 1.0 / (40.0 + 3.0j)
    assert float(torch.view_as_real(x).abs().max()) <= 1e-10 / 40.0


def test_room_for_others_stays_free():
    """Four slots would leave less than a sixteenth of the card free."""
    torch = torch_cuda()
    total = torch.cuda.mem_get_info()[1]
    shape, vec = (256, 256, 256), 16 * 256 ** 3
    announce("batch leaves room", shape)
    for free, compact in ((total // 16 + 5 * vec, True), (total // 16 + 7 * vec, False)):
        with free_bytes(free):
            b = ofd.HelmholtzBatch([shape], [(0.4,) * 3])
            assert b.compact == compact
            b.close()
