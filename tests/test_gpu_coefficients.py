"""Epilogue coefficients of the multi-RHS Dslash: up to 16 travel with the
launch, more go through a device buffer.  Both routes give the same bits on
either entry point, on two streams at once, and in a replayed graph, which keeps
the coefficients of its capture."""

import numpy as np
import pytest

import synth
from gpu_util import fields, flush, hisq, make_gauge, to_device, to_host
from layout import encode, spinor_nbytes, to_cb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s"])
def test_coefficients(cuda_device, prec):
    import torch
    H = hisq()
    dims, nmax = (6, 6, 6, 6), 19
    F, L = fields(dims)
    g = make_gauge(dims, F, L)
    nb = spinor_nbytes(prec, synth.volume(dims) // 2)
    stack = lambda par, at: to_device(np.concatenate(
        [encode(to_cb(dims, s, par), prec) for s in synth.gaussian_source(dims, 99, nmax, parity=par, index0=at)]))
    inp, y = stack(1, 20), stack(0, 60)
    diag = [0.1 + 0.037 * i for i in range(nmax)]
    want = torch.empty(nmax * nb, dtype=torch.uint8, device="cuda")
    H.dslash_multi_rhs(g, 0, prec, nmax, inp, want, diag, y)  # through the buffer
    want = to_host(want)
    entries = (H.dslash_multi_rhs, H.dslash_multi_rhs_noalloc)
    for n in (1, 2, 5, 15, 16, 17, 18):
        for fn in entries:
            flush(f"coefficients {prec} n {n} {fn.__name__}")
            out = torch.full((n * nb,), 7, dtype=torch.uint8, device="cuda")
            fn(g, 0, prec, n, inp, out, diag[:n], y)
            assert np.array_equal(to_host(out), want[:n * nb]), (n, fn.__name__)
    # two streams at once, other coefficients on each
    n = 4
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [torch.empty(n * nb, dtype=torch.uint8, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(5):
        for k, s in enumerate(streams):
            H.dslash_multi_rhs_noalloc(g, 0, prec, n, inp[k * nb:(k + n) * nb], outs[k], diag[k:k + n],
                                       y[k * nb:(k + n) * nb], stream=s)
    torch.cuda.synchronize()
    for k in range(2):
        assert np.array_equal(to_host(outs[k]), want[k * nb:(k + n) * nb]), k
    # captured, replayed with calls of other coefficients between the replays
    for fn in entries:
        flush(f"coefficients {prec} captured {fn.__name__}")
        out = torch.empty(n * nb, dtype=torch.uint8, device="cuda")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            fn(g, 0, prec, n, inp, out, list(diag[:n]), y, stream=torch.cuda.current_stream())
        for _ in range(3):
            fn(g, 0, prec, n, inp, outs[0], diag[-n:], y)
            torch.cuda.synchronize()
            out.fill_(7)
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(to_host(out), want[:n * nb]), fn.__name__
        graph.reset()
    g.close()
