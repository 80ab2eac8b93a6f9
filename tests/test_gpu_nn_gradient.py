"""The weight gradient against the FP64 oracle where the last tile of 32 sites is
ragged (6^4: 1296 sites, 648 of them even) and where it is full, with one layer
(even input and output), odd channel counts and all eight.  Bars as in
test_gpu_nn.py: BF16 operands of a few layers, 5e-2 for the gradient, 2e-2 for
the loss."""

import numpy as np
import pytest

import oracle
from oracle import nn
import synth
from gpu_util import flush, to_device
from layout import decode, encode, from_cb, rel_l2, to_cb
from test_gpu_nn import setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(6, 6, 6, 6), (4, 6, 4, 4), (8, 4, 4, 4)])
@pytest.mark.parametrize("channels", [(1, 1), (1, 3, 5, 1), (1, 8, 8, 1)])
def test_gradient(cuda_device, dims, channels):
    flush(f"gradient {dims} {channels}")
    g, net, F, L, U, ws = setup(dims, channels, seed=5, noise=0.3, scale_identity=0.5)
    vh = synth.volume(dims) // 2
    vs = synth.gaussian_source(dims, 99, 2, parity=0, index0=40)
    raw = [np.concatenate([encode(to_cb(dims, f, 0), "fp32") for f in fs])
           for fs in ([oracle.normal_op(dims, F, L, 0.3, v) for v in vs], vs)]
    loss, grad = net.loss_grad(2, to_device(raw[0]), to_device(raw[1]))
    q = lambda r, i: from_cb(dims, decode(r[i * 24 * vh:(i + 1) * 24 * vh], vh, "fp32"), 0)  # noqa: E731
    want_loss, grads = nn.loss_and_grad(dims, U, ws, [(q(raw[0], i), q(raw[1], i)) for i in range(2)])
    want = np.concatenate([w.ravel() for w in grads])
    assert abs(loss - want_loss) <= 2e-2 * want_loss
    assert rel_l2(grad, want) <= 5e-2
    net.close()
    g.close()
