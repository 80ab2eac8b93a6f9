"""Split Dslash: the hops of 64 sites over four wavefronts, for every link
storage (whole, sign and kappa rows; FP16 compresses two directions to a chunk),
plain and epilogue, with a last tile that is full and that is not, and by default
up to its largest lattice.  The sum goes through the wavefronts in the other
kernels' order, so results are compared bit for bit with them."""

import numpy as np
import pytest

import synth
from gpu_util import fields, flush, force_shape, hisq, make_gauge, to_device, to_host
from layout import encode, spinor_nbytes, to_cb
from test_gpu_pack import links

pytestmark = pytest.mark.gpu

SPLIT, PLAIN = (1, 256, 4), (1, 64, 0)


def stack(dims, prec, n, parity, at):
    return to_device(np.concatenate([encode(to_cb(dims, s, parity), prec)
                                     for s in synth.gaussian_source(dims, 99, n, parity=parity, index0=at)]))


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 6, 6, 6)])
@pytest.mark.parametrize("mode", ["whole", "sign", "kappa"])
def test_matches_plain(tmp_path, cuda_device, dims, mode):
    import torch
    H = hisq()
    F, L = links(dims, mode)
    g = make_gauge(dims, F, L, full_links=mode == "whole")
    assert g.comp_mode == {"whole": 0, "sign": 1, "kappa": 2}[mode]
    n = 3
    for prec in ("fp64", "fp32", "fp16s"):
        nb = spinor_nbytes(prec, synth.volume(dims) // 2)
        for parity in (0, 1):
            inp, y = stack(dims, prec, n, 1 - parity, 20), stack(dims, prec, n, parity, 40)
            got = {}
            for sh in (PLAIN, SPLIT):
                flush(f"split {dims} {mode} {prec} parity {parity} {sh}")
                out = torch.full((2, n * nb), 7, dtype=torch.uint8, device="cuda")
                for e in (0, 1):
                    assert force_shape(g, prec, n, e, sh, tmp_path / f"{prec}{parity}{e}{sh[2]}.jsonl") == sh
                    H.dslash_multi_rhs(g, parity, prec, n, inp, out[e], *(([0.3, 0.5, 0.7], y) if e else ()))
                got[sh] = to_host(out.reshape(-1))
            assert np.array_equal(got[SPLIT], got[PLAIN]), (prec, parity)
    g.close()


@pytest.mark.parametrize("prec,tiles", [("fp64", 256), ("fp32", 512), ("fp16s", 512)])
def test_default_limits(tmp_path, cuda_device, prec, tiles):
    """The default up to that many tiles times right-hand sides, and the same
    result on the other side of the limit."""
    import torch
    H = hisq()
    for tail, n, want in ((8, 1, SPLIT), (8, 2, None), (10, 1, None)):
        dims = (16, 16, tiles // 16, tail)
        F, L = fields(dims)
        g = make_gauge(dims, F, L, precs=(prec,))
        nb = spinor_nbytes(prec, synth.volume(dims) // 2)
        inp = stack(dims, prec, n, 1, 20)
        flush(f"split default {dims} {prec} n {n}")
        shape = H.dslash_shape(g, prec, n, 0)
        assert (shape == SPLIT) == (want == SPLIT)
        out = torch.empty(2, n * nb, dtype=torch.uint8, device="cuda")
        H.dslash_multi_rhs(g, 0, prec, n, inp, out[0])
        assert force_shape(g, prec, n, 0, SPLIT, tmp_path / f"{tail}{n}.jsonl") == SPLIT
        H.dslash_multi_rhs(g, 0, prec, n, inp, out[1])
        assert torch.equal(out[0], out[1])
        g.close()


@pytest.mark.parametrize("sloppy", ["fp64", "fp32", "fp16s", "fp16l"])
def test_solve(cuda_device, sloppy):
    """A solve of two right-hand sides of which one ends at once (zero): the
    partial sums and the skipped workgroups."""
    import torch
    H = hisq()
    dims = (4, 6, 4, 6)
    F, L = fields(dims)
    g = make_gauge(dims, F, L)
    vh = synth.volume(dims) // 2
    src = synth.gaussian_source(dims, 99, 1, parity=0)[0]
    b = to_device(np.concatenate([encode(to_cb(dims, src, 0), "fp64"), np.zeros(48 * vh, np.uint8)]))
    x = torch.zeros_like(b)
    flush(f"split solve {sloppy}")
    st = H.cg_solve(g, 0.2, 2, b, x, H.solver_params(sloppy_prec=sloppy, tol=1e-10))
    t, r = torch.empty_like(b), torch.empty_like(b)
    H.dslash_multi_rhs(g, 1, "fp64", 2, x, t)
    H.dslash_multi_rhs(g, 0, "fp64", 2, t, r, [4 * 0.2 ** 2] * 2, x)
    d, bb = (to_host(v)[:48 * vh].view(np.float64) for v in (r, b))
    assert np.linalg.norm(d - bb) <= 2e-10 * np.linalg.norm(bb)
    assert not to_host(x)[48 * vh:].any()
    g.close()
