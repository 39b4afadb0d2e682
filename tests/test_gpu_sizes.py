"""Launches of more work items than one dimension of a grid may have."""
import pytest

import paper_2503_01873_amd as P
from gpu_harness import f32

pytestmark = pytest.mark.gpu


def test_keys_of_four_million_heads_are_shifted():
    """2^22 key tiles of a single key each: 2^32 work items for the key blocks alone."""
    import torch
    B, H, d, scale = 1 << 11, 1 << 11, 64, 0.125
    k = torch.empty((B, H, 1, d), dtype=torch.float16, device="cuda:0").normal_()
    out = torch.zeros_like(k)
    beta = 0.9375
    P.pasa_shift_keys(k, out, B, H, 1, d, beta, f32(scale))
    torch.cuda.synchronize()
    for b in (0, B // 2, B - 1):
        want = ((k[b].double() - beta * k[b].double()) * scale).half()      # a tile's mean is its only key; every step is exact
        assert torch.equal(out[b], want)
    del k, out
    torch.cuda.empty_cache()
