"""GPU smearing on the lattices where its field tiles and site sweep have
remainders: a last tile of fewer than 64 sites, columns narrower than the
others in y or z, extents below a column's side, and blocks of 64 and of 256
threads.

Tolerance: FP64 on both sides, 1e-12 absolute on entries of size ~1 as in
test_gpu_smear.py (at most ~2^-53 times a few thousand products per entry)."""

import numpy as np
import pytest

import synth
from gpu_util import flush, hisq, to_device, to_host
from oracle import smear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(6, 6, 6, 6), (4, 4, 4, 4), (6, 4, 10, 14), (48, 8, 4, 4), (20, 14, 12, 4)])
def test_smear_remainders(cuda_device, dims):
    import torch
    flush(f"smear sweep {dims}")
    U = synth.thin_links(dims, 131, 0.5)
    t = to_device(np.ascontiguousarray(U))
    fat, lng = torch.empty_like(t), torch.empty_like(t)
    hisq().smear_links(dims, t, fat, lng, antiperiodic_t=True)
    assert np.array_equal(to_host(t), U)  # the input is only read
    Fo, Lo = smear.hisq_smear(dims, U, antiperiodic_t=True)
    assert np.abs(to_host(fat) - Fo).max() < 1e-12
    assert np.abs(to_host(lng) - Lo).max() < 1e-12


def test_smear_remainders_large_blocks(cuda_device):
    """32 x 10 x 22 x 38 = 267520 sites: blocks of 256 threads, a last one that
    is not full, columns of 7 x 7 rows with narrower last ones.  The corners,
    the last column's sites and random ones against the single-site oracle; every
    site against unitarity of the Naik links (and so of W)."""
    import torch
    dims = (32, 10, 22, 38)
    flush(f"smear sweep {dims}")
    U = synth.thin_links(dims, 132, 0.5)
    t = to_device(np.ascontiguousarray(U))
    fat, lng = torch.empty_like(t), torch.empty_like(t)
    hisq().smear_links(dims, t, fat, lng)
    F, L = to_host(fat), to_host(lng)
    V = synth.volume(dims)
    LL = np.einsum("vmba,vmbc->vmac", L.conj(), L)
    assert np.abs(LL - np.eye(3) / 576).max() < 1e-13 / 576
    lex = lambda x, y, z, t_: x + 32 * (y + 10 * (z + 22 * t_))  # noqa: E731
    sites = [0, V - 1, lex(0, 9, 21, 0), lex(31, 7, 21, 37), lex(17, 9, 20, 19)]
    sites += list(np.random.default_rng(6).choice(V, 5, replace=False))
    for s_ in sites:
        f, l = smear.hisq_smear_at(dims, U, int(s_))
        assert np.abs(F[s_] - f).max() < 1e-12 and np.abs(L[s_] - l).max() < 1e-12, s_
