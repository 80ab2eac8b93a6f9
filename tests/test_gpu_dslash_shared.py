"""Shared-link multi-RHS Dslash: every (R, W) that is built, ragged numbers of
right-hand sides (a wavefront with fewer than R, or with none), a last tile
that is not full, whole and compressed links, plain and epilogue, through the
default shapes and forced ones.  The arithmetic per site is the other kernels',
in the same order, so plain results are compared bit for bit with one
right-hand side at a time; the oracle judges those elsewhere, and here once."""

import numpy as np
import pytest

import oracle
import synth
from gpu_util import fields, flush, force_shape, hisq, make_gauge, to_device, to_host
from layout import decode, encode, from_cb, rel_l2, spinor_nbytes, to_cb

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-13, "fp32": 1e-6, "fp16s": 2e-3}
WAVES = {2: 1, 4: 2, 3: 3}  # bits 24-25 of the order
BUILT = [(1, 2), (1, 3), (1, 4), (2, 3), (2, 4), (3, 3), (3, 4), (4, 4)]


def shape(r, w):
    return (r, 64 * w, 2 | WAVES[w] << 24)


def singles(H, g, parity, prec, n, inp, nb):
    """The right-hand sides one at a time (one per thread)."""
    import torch
    out = torch.empty(n * nb, dtype=torch.uint8, device="cuda")
    for i in range(n):
        H.dslash_eo(g, parity, prec, inp[i * nb:(i + 1) * nb], out[i * nb:(i + 1) * nb])
    return to_host(out)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s"])
@pytest.mark.parametrize("full", [False, True])
def test_every_shape_matches_single(tmp_path, cuda_device, prec, full):
    import torch
    H = hisq()
    dims = (6, 6, 6, 6)  # Vh = 648: ten tiles and 8 sites
    F, L = fields(dims)
    g = make_gauge(dims, F, L, full_links=full)
    vh = synth.volume(dims) // 2
    nb = spinor_nbytes(prec, vh)
    nmax = 17
    srcs = synth.gaussian_source(dims, 99, nmax, parity=1, index0=20)
    raw = np.concatenate([encode(to_cb(dims, s, 1), prec) for s in srcs])
    inp = to_device(raw)
    want = singles(H, g, 0, prec, nmax, inp, nb)
    diag = [0.1 + 0.01 * i for i in range(nmax)]
    for r, w in BUILT:
        for n in sorted({r * (w - 1) + 1, r * w, 17}):
            flush(f"shared {prec} full {full} R {r} W {w} n {n}")
            sh = shape(r, w)
            assert force_shape(g, prec, n, 0, sh, tmp_path / f"p{r}{w}{n}.jsonl") == sh
            out = torch.full((n * nb,), 7, dtype=torch.uint8, device="cuda")
            H.dslash_multi_rhs(g, 0, prec, n, inp, out)
            assert np.array_equal(to_host(out), want[:n * nb]), (r, w, n)
            # epilogue: diag y - D in with y of the output parity, against the same with one RHS
            assert force_shape(g, prec, n, 1, sh, tmp_path / f"e{r}{w}{n}.jsonl") == sh
            y = inp[:n * nb]
            H.dslash_multi_rhs(g, 0, prec, n, inp, out, diag[:n], y)
            got = to_host(out)
            one = torch.empty(nb, dtype=torch.uint8, device="cuda")
            for i in (0, n - 1):
                H.dslash_multi_rhs(g, 0, prec, 1, inp[i * nb:(i + 1) * nb], one, [diag[i]], y[i * nb:(i + 1) * nb])
                assert np.array_equal(got[i * nb:(i + 1) * nb], to_host(one)), (r, w, n, i)
    got = want.reshape(nmax, -1)
    for i in (0, nmax - 1):
        chi = from_cb(dims, decode(raw[i * nb:(i + 1) * nb], vh, prec), 1)
        assert rel_l2(decode(got[i], vh, prec), to_cb(dims, oracle.dslash(dims, F, L, chi, 0), 0)) <= TOL[prec]
    g.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 6, 6, 6), (20, 18, 14, 10), (8, 8, 8, 64)])
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp16s"])
def test_default_shapes(cuda_device, dims, prec):
    """The default shape of every number of right-hand sides from 1 to 19 and 33
    (few and many wavefronts, tiles per thread, shared, more than one workgroup
    per tile) gives the single right-hand side's bits."""
    import torch
    H = hisq()
    F, L = fields(dims)
    g = make_gauge(dims, F, L)
    vh = synth.volume(dims) // 2
    nb = spinor_nbytes(prec, vh)
    nmax = 33
    base = synth.gaussian_source(dims, 99, 3, parity=1)
    enc = [encode(to_cb(dims, (1 + 0.1 * i) * base[i % 3], 1), prec) for i in range(nmax)]
    inp = to_device(np.concatenate(enc))
    want = singles(H, g, 0, prec, nmax, inp, nb)
    for n in list(range(1, 20)) + [33]:
        out = torch.empty(n * nb, dtype=torch.uint8, device="cuda")
        H.dslash_multi_rhs(g, 0, prec, n, inp, out)
        assert np.array_equal(to_host(out), want[:n * nb]), (n, H.dslash_shape(g, prec, n, 0))
    g.close()


@pytest.mark.parametrize("sloppy", ["fp64", "fp32", "fp16s", "fp16l"])
@pytest.mark.parametrize("n", [3, 7, 18])
def test_batched_solve(cuda_device, sloppy, n):
    """A solve whose batch shrinks (different norms of the start) through the
    default shapes: every solution on the oracle's true residual."""
    import torch
    H = hisq()
    dims = (12, 12, 10, 8)  # 90 tiles: shared from 12 right-hand sides in FP32, from 2 in FP64
    F, L = fields(dims)
    g = make_gauge(dims, F, L)
    vh = synth.volume(dims) // 2
    mass = 0.2
    b = synth.gaussian_source(dims, 55, n, parity=0)
    bd = to_device(np.concatenate([encode(to_cb(dims, (10.0 ** (i % 3)) * v, 0), "fp64") for i, v in enumerate(b)]))
    x = torch.zeros_like(bd)
    rc, st = H.cg_solve(g, mass, n, bd, x, H.solver_params(sloppy_prec=sloppy))
    assert rc == 0, st
    xs = to_host(x).reshape(n, -1)
    for i in (0, n // 2, n - 1):
        xf = from_cb(dims, decode(xs[i], vh, "fp64"), 0)
        assert oracle.true_residual(dims, F, L, mass, 10.0 ** (i % 3) * b[i], xf) <= 1e-10
    g.close()
