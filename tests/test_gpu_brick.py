"""The brick kernel that small grids run (no launch-table entry): axes at its
smallest size, axes that fill no tile, planes left over in z, one and four
planes per brick, against the oracle and bitwise against the marched tiles
(same operations in the same order per point)."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import fd, poisson
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu

# up to 2^17 points: one plane per brick; above: four (nz % 4 = 0, 1, 2, 3)
SHAPES = [(10, 10, 10), (11, 13, 10), (12, 10, 129), (10, 300, 11), (17, 64, 65), (50, 53, 61), (51, 64, 64), (53, 41, 70),
          (44, 20, 200)]
ELEM = {"f64": 8, "f32": 4, "c128": 16, "c64": 8}


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", ["f64", "f32", "c128", "c64"])
def test_apply(shape, dtype):
    torch = torch_cuda()
    announce("brick", shape, dtype)
    h = (0.4, 0.45, 0.5)
    rng = np.random.default_rng(sum(shape))
    cx = dtype in ("c128", "c64")
    x = rng.normal(size=shape) + (1j * rng.normal(size=shape) if cx else 0.0)
    tdt = {"f64": torch.float64, "f32": torch.float32, "c128": torch.complex128, "c64": torch.complex64}[dtype]
    xd = to_dev(x, tdt)
    y0 = to_dev(rng.normal(size=shape) + (0j if cx else 0.0), tdt)
    ya, yb = torch.full_like(xd, float("nan")), y0.clone()
    ofd.fd_laplacian_apply(xd, ya, h)
    ofd.fd_laplacian_apply(xd, yb, h, alpha=-0.7, beta=1.3)
    xin = to_host(xd).astype(np.complex128 if cx else np.float64)
    ref = fd.laplacian(xin, h, 6)
    w = np.concatenate([fd.weights(6, hh) for hh in h])
    tol = (1e-14 if dtype in ("f64", "c128") else 2e-6) * np.abs(w).sum() * np.abs(xin).max()
    assert np.abs(to_host(ya) - ref).max() <= tol
    try:
        ofd.set_stencil_config(shape, ELEM[dtype], 2)
        ma, mb = torch.full_like(xd, float("nan")), y0.clone()
        ofd.fd_laplacian_apply(xd, ma, h)
        ofd.fd_laplacian_apply(xd, mb, h, alpha=-0.7, beta=1.3)
        assert torch.equal(ya, ma) and torch.equal(yb, mb)
    finally:
        ofd.set_stencil_config(shape, ELEM[dtype], -1)


@pytest.mark.parametrize("mode", [ofd.PLAIN_F64, ofd.REFINED_F32])
@pytest.mark.parametrize("shape", [(10, 11, 12), (13, 40, 17), (53, 41, 70)])
def test_solve(shape, mode):
    """The two-array loader and the reductions of the CG passes on bricks."""
    torch_cuda()
    announce("brick solve", shape, mode)
    h = (0.4, 0.45, 0.5)
    g = np.random.default_rng(7).normal(size=shape)
    s = ofd.PoissonSolver(shape, h, 6, mode)
    phi = to_dev(np.zeros(shape))
    s.solve(to_dev(g), phi, 1e-10)
    assert poisson.residual(to_host(phi), g - g.mean(), h) <= 1e-10
    s.close()
