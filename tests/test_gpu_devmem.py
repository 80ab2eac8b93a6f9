"""Device memory that the library keeps between handles and calls: a handle or
a workspace on a block that held other data gives the same bits as one on
fresh memory, and threads with streams of their own do not disturb each other.

The comparisons are bit for bit: the same kernels run on the same inputs."""

import threading

import numpy as np
import pytest

import synth
from gpu_util import fields, flush, hisq, make_gauge, to_device, to_host
from layout import encode, spinor_nbytes, to_cb

pytestmark = pytest.mark.gpu

DIMS = (10, 6, 4, 8)  # Vh = 960: the last tile of every link buffer is full of padding


def outputs(H, g, mass=0.2, stream=None, chunk=32):
    """A solve, a rational function and a Dslash of every precision, as bytes."""
    import torch
    vh = synth.volume(DIMS) // 2
    b = to_device(encode(to_cb(DIMS, synth.gaussian_source(DIMS, 7, 1, parity=0)[0], 0), "fp64"))
    got = []
    x = torch.empty_like(b)
    for sloppy in ("fp64", "fp32"):
        H.cg_solve(g, mass, 1, b, x, H.solver_params(sloppy_prec=sloppy, graph_chunk=chunk), stream=stream)
        got.append(to_host(x))
    H.rational_apply(g, mass, 0.5, [0.3, 0.2, 0.1], [0.01, 0.1, 1.0], b, x,
                     H.solver_params(sloppy_prec="fp32", graph_chunk=chunk), stream=stream)
    got.append(to_host(x))
    odd = synth.gaussian_source(DIMS, 8, 1, parity=1)[0]
    for prec in ("fp64", "fp32", "fp16s"):
        inp = to_device(encode(to_cb(DIMS, odd, 1), prec))
        out = torch.empty(spinor_nbytes(prec, vh), dtype=torch.uint8, device="cuda")
        H.dslash_eo(g, 0, prec, inp, out, stream=stream)
        torch.cuda.synchronize()
        got.append(to_host(out))
    return got


def test_reused_blocks_give_the_same_bits(cuda_device):
    H = hisq()
    F, L = fields(DIMS)
    flush("devmem: fresh handle")
    g = make_gauge(DIMS, F, L)
    want = outputs(H, g)
    g.close()
    for k in range(3):
        flush(f"devmem: dirty blocks {k}")
        d = make_gauge(DIMS, 50.0 * (k + 1) * F, 40.0 * L)  # other values on the same blocks
        d.close()
        g = make_gauge(DIMS, F, L)
        for a, b in zip(want, outputs(H, g)):
            assert np.array_equal(a, b)
        g.close()


def test_threads_and_streams(cuda_device):
    """Three threads make, use and free handles at once (eager launches: a device
    synchronisation, as of freeing a handle, is not allowed while another thread
    captures a graph)."""
    import torch
    H = hisq()
    F, L = fields(DIMS)
    g = make_gauge(DIMS, F, L)
    want = outputs(H, g, chunk=0)
    g.close()
    seen = []

    def work():
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for _ in range(3):
                    h = make_gauge(DIMS, F, L)
                    seen.extend(np.array_equal(a, b) for a, b in zip(want, outputs(H, h, stream=s, chunk=0)))
                    h.close()
        except Exception as e:  # to the main thread
            seen.append(e)

    flush("devmem: three threads")
    threads = [threading.Thread(target=work) for _ in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(100)
    assert seen == [True] * (3 * 3 * len(want))
