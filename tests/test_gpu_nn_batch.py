"""Training batches whose samples go through the network together: ragged
lattices, one layer and several, a batch that needs more than one group, and the
growth of the buffers between calls.

A batch repeated 8 times has the same loss and gradient: the scale 2 / (B |v|^2)
changes by a power of two, so every rounding of the backward pass scales with
it, and what is left is the FP64 sum of 8 times as many terms (1e-12)."""

import numpy as np
import pytest

import synth
from gpu_util import fields, flush, hisq, make_gauge, to_device
from layout import encode, to_cb

pytestmark = pytest.mark.gpu


def setup(dims, channels, n, seed=3):
    H = hisq()
    F, L = fields(dims)
    g = make_gauge(dims, F, L, precs=("fp32",))
    U = np.ascontiguousarray(synth.thin_links(dims, 99, 0.5))
    H.gauge_set_thin(g, to_device(U))
    r = np.random.default_rng(seed)
    nw = sum(9 * a * b for a, b in zip(channels[:-1], channels[1:]))
    net = H.Net(g, channels, 0.2 * (r.standard_normal(nw) + 1j * r.standard_normal(nw)))
    v = synth.gaussian_source(dims, 31, n, parity=0)
    w = synth.gaussian_source(dims, 31, n, parity=0, index0=50)
    enc = lambda fs: np.concatenate([encode(to_cb(dims, f, 0), "fp32") for f in fs])  # noqa: E731
    return g, net, enc(w), enc(v)


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 6, 6, 6), (10, 6, 4, 8)])
@pytest.mark.parametrize("channels", [(1, 1), (1, 5, 1), (1, 8, 3, 1)])
def test_repeated_batch(cuda_device, dims, channels):
    flush(f"nn batch {dims} {channels}")
    g, net, av, v = setup(dims, channels, 3)
    loss, grad = net.loss_grad(3, to_device(av), to_device(v))
    loss8, grad8 = net.loss_grad(24, to_device(np.tile(av, 8)), to_device(np.tile(v, 8)))
    again, gagain = net.loss_grad(3, to_device(av), to_device(v))  # with the larger buffers
    assert again == loss and np.array_equal(gagain, grad)
    assert abs(loss8 - loss) <= 1e-12 * loss
    assert np.linalg.norm(grad8 - grad) <= 1e-12 * np.linalg.norm(grad)
    net.close()
    g.close()


def test_more_than_one_group(cuda_device):
    """4^4: 512 MiB hold about 1300 samples; 200 x 8 are two groups."""
    dims = (4, 4, 4, 4)
    g, net, av, v = setup(dims, (1, 8, 8, 1), 200)
    loss, grad = net.loss_grad(200, to_device(av), to_device(v))
    loss8, grad8 = net.loss_grad(1600, to_device(np.tile(av, 8)), to_device(np.tile(v, 8)))
    assert abs(loss8 - loss) <= 1e-12 * loss
    assert np.linalg.norm(grad8 - grad) <= 1e-12 * np.linalg.norm(grad)
    net.close()
    g.close()
