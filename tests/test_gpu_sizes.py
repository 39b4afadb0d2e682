"""Launches of more work items, and lists of more rows, than 32 bits count."""
import pytest

import paper_2503_01873_amd as P
from gpu_harness import f32, plan_of

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


def test_rows_of_two_million_heads_on_one():
    """2^24 query rows that share the keys of one KV head, 4 GiB of them: the bits of the same rows a thousand heads at a time."""
    import torch
    Hq, Nq, N, d, scale = 1 << 21, 8, 64, 128, f32(128 ** -0.5)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    q = torch.empty((1, Hq, Nq, d), dtype=torch.float16, device="cuda:0").normal_(generator=gen)
    k, v = (torch.empty((1, 1, N, d), dtype=torch.float16, device="cuda:0").normal_(generator=gen) for _ in range(2))
    wsb = P.pasa_attn_fwd_workspace_min(1, 1, N, d)
    ws = torch.empty(wsb, dtype=torch.uint8, device="cuda:0")
    stream = torch.cuda.current_stream()
    P.pasa_prepare_kv(k, v, 1, 1, N, d, scale, ws, wsb, stream)

    def rows_of(x):
        o = torch.full_like(x, float("nan"))
        H = x.shape[1]
        assert plan_of(P.MIXED, 1, H, 1, Nq, N - Nq, N, d, True, workspace_bytes=wsb) == ("rows", 1)
        P.pasa_attn_fwd_chunk(x, o, 1, H, 1, Nq, N - Nq, N, d, True, scale, ws, wsb, stream)
        torch.cuda.synchronize()
        return o

    o = rows_of(q)
    for h in (0, Hq // 2, Hq - 1024):
        part = rows_of(q[:, h:h + 1024].contiguous())
        assert bool(torch.isfinite(part).all()) and float(part.abs().max()) > 0.5
        assert torch.equal(o[:, h:h + 1024], part), h
    del q, o
    torch.cuda.empty_cache()
