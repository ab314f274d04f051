"""The network's convolution and weight-gradient bricks on grids where their
choice changes (large bricks with one, two or three output tiles, small bricks,
z columns of one, two and four bricks) and where a level is shorter than a
brick: one application and the weight gradients against the FP64 reference, in
the FP32 mode element by element."""
import numpy as np
import pytest

import paper_1412_8250_amd as ofd
from oracle import nn as onn
from tests.gpu_util import announce, to_dev, to_host, torch_cuda

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(8, 8, 8), (8, 16, 40), (24, 8, 48), (32, 24, 56)])
def test_fp32_mode_matches_reference(shape):
    torch = torch_cuda()
    announce("nn bricks", shape)
    h = (0.4, 0.4, 0.4)
    rng = np.random.default_rng(6)
    W = {k: w.astype(np.float32) for k, w in onn.init_weights(rng).items()}
    g, phi = rng.normal(size=shape), rng.normal(size=shape)
    net = ofd.Network(1)
    net.set_precision(True)
    net.set_weights(W)
    W64 = {k: w.astype(np.float64) for k, w in W.items()}
    rms = np.sqrt((g * g).mean())
    out, cache = onn.forward(W64, g / rms)
    o = to_dev(np.zeros(shape))
    net.forward(to_dev(g), o, h)
    ref = rms * out
    # FP32 activations: the stated bound of the element-wise check, 1e-5 of the tensor's largest
    assert np.abs(to_host(o) - ref).max() <= 1e-5 * np.abs(ref).max()
    t = phi / (0.4 ** 2 * rms)
    _, dout = onn.loss(out, t)
    grads = onn.backward(W64, cache, dout)
    net.gradients(to_dev(g), to_dev(phi), h)
    got = net.get_weights(gradients=True)
    for name, ref in grads.items():
        assert np.abs(got[name] - ref).max() <= 1e-5 * np.abs(ref).max(), name
    back = net.get_weights()
    assert all(np.array_equal(back[k], W[k]) for k in W)
    net.close()


@pytest.mark.parametrize("shape", [(64, 32, 32), (16, 128, 32)])
def test_bf16_application_at_both_brick_sizes(shape):
    """Level 0 on large bricks, the coarse levels on small ones (BF16)."""
    torch_cuda()
    announce("nn bricks bf16", shape)
    rng = np.random.default_rng(7)
    W = {k: w.astype(np.float32) for k, w in onn.init_weights(rng).items()}
    g = rng.normal(size=shape)
    net = ofd.Network(1)
    net.set_weights(W)
    o = to_dev(np.zeros(shape))
    net.forward(to_dev(g), o, (0.4,) * 3)
    rms = np.sqrt((g * g).mean())
    ref = rms * onn.forward({k: w.astype(np.float64) for k, w in W.items()}, g / rms)[0]
    # 12 u sqrt(D) of the tensor's largest, u = 2^-8 per stored value, D = 17 stages
    assert np.abs(to_host(o) - ref).max() <= 12 * 2.0 ** -8 * np.sqrt(17.0) * np.abs(ref).max()
    net.close()
