"""Splitting a sequence at multiples of 32 rows gives the bits of the whole call wherever the keys are swept unsplit, whatever
kernel the whole is planned on."""
import numpy as np
import pytest

import paper_2503_01873_amd as P
from gpu_harness import f32, gpu_attn, gpu_attn_chunks, plan_of

pytestmark = pytest.mark.gpu

# B, Hq, Hkv, N, d, causal, pieces (rows of each), kernel of the whole (None: any)
CASES = [
    (1, 28, 4, 777, 128, True, (256, 256, 256, 9), "rows"),          # the last piece is shorter than a wavefront's rows
    (1, 28, 4, 1024, 128, True, (32, 96, 512, 384), "halves"),
    (1, 28, 4, 1100, 128, True, (512, 512, 64, 12), "halves"),
    (1, 28, 4, 2048, 128, True, (1024, 992, 32), "halves"),
    (1, 28, 4, 900, 128, False, (33, 500, 367), "halves"),
    (1, 28, 4, 4096, 128, True, (2048, 2048), "fwd"),                # 224 workgroups of 256 rows each: not split
    (14, 6, 6, 1000, 64, True, (32, 480, 480, 8), "fwd4"),
    (14, 6, 6, 1000, 64, False, (100, 900), "fwd4"),
    (14, 16, 16, 2176, 64, True, (1024, 1152), None),                # more than 2048 keys
    (1, 1, 1, 2048, 64, True, (64, 1024, 960), None),
]


@pytest.mark.parametrize("variant", [P.MIXED, P.S16, P.DIRECT])
@pytest.mark.parametrize("B,Hq,Hkv,N,d,causal,pieces,kernel", CASES)
def test_pieces_have_the_bits_of_the_whole(B, Hq, Hkv, N, d, causal, pieces, kernel, variant):
    if kernel is not None and variant != P.S16:
        assert plan_of(variant, B, Hq, Hkv, N, 0, N, d, causal)[0] == kernel
    rng = np.random.default_rng(N + B)
    q = rng.standard_normal((B, Hq, N, d)).astype(np.float16)
    k = (rng.standard_normal((B, Hkv, N, d)) + 2).astype(np.float16)
    v = rng.standard_normal((B, Hkv, N, d)).astype(np.float16)
    scale = f32(d ** -0.5)
    whole, _ = gpu_attn(q, k, v, causal, scale, variant)
    assert np.isfinite(whole).all()
    first, chunks = 0, []
    for n in pieces:
        chunks.append((first, n, first))
        first += n
    assert first == N
    parts = gpu_attn_chunks(q, k, v, causal, scale, chunks, variant=variant)
    for at, n, _ in chunks:
        a, b = whole[:, :, at:at + n], parts[:, :, at:at + n]
        assert a.tobytes() == b.tobytes(), (at, n, int((a != b).sum()))
