"""Packed links where the packing has remainders: Vh no multiple of 64 (a last
tile that is not full), every layout (whole, sign, complex factor), subsets of
the precisions, and links that start 8 bytes off a 16-byte boundary.

Tolerances as for the Dslash on other lattices: 1e-13 (FP64), 1e-6 (FP32),
3e-3 (FP16S, end to end)."""

import numpy as np
import pytest

import oracle
import synth
from gpu_util import fields, flush, hisq, to_device, to_host
from layout import decode, encode, from_cb, rel_l2, spinor_nbytes, to_cb

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-13, "fp32": 1e-6, "fp16s": 3e-3}


def links(dims, mode):
    F, L = fields(dims)
    if mode == "kappa":  # positive multiples of U(3) matrices
        V = synth.volume(dims)
        ph = np.exp(1j * np.random.default_rng(3).uniform(0, 6.28, (V, 4, 1, 1)))
        L = L * ph * 0.0417
    return F, L


def at_offset(U, off):
    """Device copy of U that starts `off` bytes into a buffer; its pointer."""
    import torch
    raw = np.ascontiguousarray(U).view(np.float64).ravel()
    buf = torch.empty(raw.size + 2, dtype=torch.float64, device="cuda")
    v = buf[off // 8:off // 8 + raw.size]
    v.copy_(torch.from_numpy(raw))
    return v


@pytest.mark.parametrize("dims", [(6, 6, 6, 6), (4, 4, 4, 4), (4, 6, 10, 6), (10, 6, 4, 8)])
@pytest.mark.parametrize("mode", ["whole", "sign", "kappa"])
@pytest.mark.parametrize("precs", [("fp64", "fp32", "fp16s"), ("fp32",), ("fp16s",)])
def test_packed_remainders(cuda_device, dims, mode, precs):
    import torch
    flush(f"pack {dims} {mode} {precs}")
    H = hisq()
    F, L = links(dims, mode)
    off = 8 if dims == (6, 6, 6, 6) else 0
    g = H.Gauge(dims, at_offset(F, off), at_offset(L, off), precs, full_links=mode == "whole")
    assert g.comp_mode == {"whole": 0, "sign": 1, "kappa": 2}[mode]
    vh = synth.volume(dims) // 2
    for prec in precs:
        for parity in (0, 1):
            src = synth.gaussian_source(dims, 99, 1, parity=1 - parity)[0]
            raw = encode(to_cb(dims, src, 1 - parity), prec)
            out = torch.empty(spinor_nbytes(prec, vh), dtype=torch.uint8, device="cuda")
            H.dslash_eo(g, parity, prec, to_device(raw), out)
            chi = from_cb(dims, decode(raw, vh, prec), 1 - parity)
            want = to_cb(dims, oracle.dslash(dims, F, L, chi, parity), parity)
            assert rel_l2(decode(to_host(out), vh, prec), want) <= TOL[prec], (prec, parity)
    g.close()
