"""Device memory between handles: a destroyed handle's blocks go to the next one
without a new allocation, and hisq_release_memory gives them back."""

import pytest

from gpu_util import fields, hisq, make_gauge

pytestmark = pytest.mark.gpu

DIMS = (16, 16, 16, 16)  # 256 MB of links in the three precisions


def free_bytes():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()  # the links that torch held
    return torch.cuda.mem_get_info()[0]


def test_blocks_are_reused_and_given_back(cuda_device):
    H = hisq()
    F, L = fields(DIMS)
    make_gauge(DIMS, F, L).close()  # code objects and the runtime's own memory are there
    H.release_memory()
    start = free_bytes()
    g = make_gauge(DIMS, F, L)
    held = start - free_bytes()
    links = g.device_bytes()
    assert held >= links > 1 << 27
    g.close()
    assert start - free_bytes() >= links  # kept
    for _ in range(3):
        g = make_gauge(DIMS, F, L)
        assert start - free_bytes() <= held + (1 << 24)  # on the same blocks
        g.close()
    freed = H.release_memory()
    assert links <= freed <= held
    assert start - free_bytes() <= held - links
    assert H.release_memory() == 0
