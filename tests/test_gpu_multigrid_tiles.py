"""The multigrid cycle's two kernels per level on grids where their tiling can
go wrong: axes that fill no tile or z chunk, axes of two points (every
neighbour is an image of the point's own pair), long thin boxes, and coarsest
grids of every parity; against the reference cycle value by value."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import multigrid
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

SHAPES = [(32, 18, 30), (2, 32, 20), (20, 2, 18), (18, 26, 2), (16, 48, 176), (96, 8, 40), (88, 72, 40), (52, 36, 60)]

# FP64 levels: rounding of about 40 operations per value through every level;
# FP32 levels: the same in single precision
TOL = {ofd.MULTIGRID_F64: 1e-12, ofd.MULTIGRID: 2e-6}


@pytest.mark.parametrize("mode", [ofd.MULTIGRID_F64, ofd.MULTIGRID])
@pytest.mark.parametrize("shape", SHAPES)
def test_real_cycle_on_odd_tiles(shape, mode):
    torch = torch_cuda()
    announce("mg tiles", shape, mode)
    h = (0.45, 0.4, 0.5)
    r = np.random.default_rng(3).normal(size=shape)
    s = ofd.PoissonSolver(shape, h, 6, mode)
    rd = to_dev(r)
    z = torch.full_like(rd, float("nan"))
    s.apply_preconditioner(rd, z)
    ref = multigrid.vcycle(r, h, 0.0).real
    assert np.abs(to_host(z) - ref).max() <= TOL[mode] * np.abs(ref).max()
    s.close()


@pytest.mark.parametrize("kind", [ofd.PRECOND_MULTIGRID_F64, ofd.PRECOND_MULTIGRID])
@pytest.mark.parametrize("shape", SHAPES)
def test_complex_cycle_on_odd_tiles(shape, kind):
    torch = torch_cuda()
    announce("mg tiles complex", shape, kind)
    h = (0.45, 0.4, 0.5)
    rng = np.random.default_rng(4)
    r = rng.normal(size=shape) + 1j * rng.normal(size=shape)
    b = ofd.HelmholtzBatch([shape] * 3, [h] * 3, 6, ofd.C128)
    b.set_preconditioner(kind)
    rd = to_dev(r)
    z = torch.full_like(rd, complex("nan"))
    kap = 0.235 - 0.924j
    b.apply_preconditioner(2, kap, rd, z)
    ref = multigrid.vcycle(r, h, kap)
    tol = TOL[ofd.MULTIGRID if kind == ofd.PRECOND_MULTIGRID else ofd.MULTIGRID_F64]
    assert np.abs(to_host(z) - ref).max() <= tol * np.abs(ref).max()
    b.close()
