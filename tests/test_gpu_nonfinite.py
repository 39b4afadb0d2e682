"""Scores beyond the range of their type on every kernel: a row that sees such a key comes out as NaN, as in the oracle, and
is never finite with some of its keys left out.  A row that sees a single key tile needs no pseudo-average, so a score that
overflowed to -inf only takes its own weight there.

Two sources: an infinite key (bf16 beyond 65504 becomes one), whose tile's mean and with it every K' of the tile is infinite in
that channel; and, with S' rounded to fp16 (S16), finite inputs whose score is below -65520, which makes the tile's
pseudo-average -inf."""
import numpy as np
import pytest

import paper_2503_01873_amd as P
from oracle import pasa_oracle as po
from gpu_harness import bf16_bits, compare, f32, gpu_attn, gpu_attn_chunks, plan_of, VARIANT_NAME

pytestmark = pytest.mark.gpu

BETA = po.default_beta()
POLICY = {P.MIXED: po.MIXED, P.S16: po.PARTIAL16}


def _check(o, q, k, v, scale, causal, variant, row0, nan_from, kernel, checked_to=None):
    """Rows of one head at positions row0 ..: NaN from position nan_from on, before it the oracle's values.  The oracle sees
    the same NaN rows (its DIRECT form cannot be asked: it takes the largest finite score of every tile)."""
    pos = row0 + np.arange(len(q))
    want = (pos >= nan_from)[:, None] & np.ones(q.shape[1], bool)
    if variant != P.DIRECT:
        with np.errstate(invalid="ignore"):
            ref = po.pasa_rows(q, k, v, scale, causal, BETA, 128, POLICY[variant], row0)
        assert np.array_equal(np.isnan(ref), want)
    else:
        n = min(len(k), nan_from)
        ref = po.direct_rows(q[pos < n], k[:n], v[:n], scale, causal, BETA, 128, po.MIXED, row0) if (pos < n).any() else q[:0]
    assert np.array_equal(np.isnan(o), want), (kernel, VARIANT_NAME[variant], np.unique(np.nonzero(np.isnan(o) != want)[0])[:8])
    # Where S' is rounded, single outputs differ at a dominant key whose score straddles a rounding boundary; and in the tile of an
    # overflowing key the scores are near 780 (its share of the mean), where a step of fp16 is 0.5 and moves a weight by e^0.5:
    # there only finiteness is asked for.
    ok = pos < (nan_from if checked_to is None else checked_to)
    if ok.any():
        c = compare(o[ok], ref[:ok.sum()])
        assert (c["maxabs"] <= 2e-3) if variant != P.S16 else (c["p999"] <= 2e-3)


def _inputs(rng, B, Hq, Hkv, Nq, N, d):
    return (rng.standard_normal((B, Hq, Nq, d)).astype(np.float16), (rng.standard_normal((B, Hkv, N, d)) + 1).astype(np.float16),
            rng.standard_normal((B, Hkv, N, d)).astype(np.float16))


# ------------------------------------------------------------------ an infinite key

@pytest.mark.parametrize("variant", [P.MIXED, P.DIRECT, P.S16])
@pytest.mark.parametrize("d,N,inf_key", [(64, 300, 200), (128, 300, 250), (128, 200, 199), (64, 500, 100)])
def test_infinite_key_few_rows(d, N, inf_key, variant):
    rng = np.random.default_rng(N + inf_key)
    q, k, v = _inputs(rng, 1, 2, 2, N, N, d)
    k[0, :, inf_key, 5] = np.inf
    scale = f32(d ** -0.5)
    assert plan_of(variant, 1, 2, 2, N, 0, N, d, True) == ("rows", 1)
    o, _ = gpu_attn(q, k, v, True, scale, variant)
    for h in range(2):
        _check(o[0, h], q[0, h], k[0, h], v[0, h], scale, True, variant, 0, inf_key // 128 * 128, "rows")


@pytest.mark.parametrize("variant", [P.MIXED, P.DIRECT, P.S16])
def test_infinite_key_decoding_step(variant):
    """The key lies past the row's position, in its tile; the keys are swept in pieces."""
    rng = np.random.default_rng(12)
    N, d, scale = 6000, 128, f32(128 ** -0.5)
    q, k, v = _inputs(rng, 1, 4, 2, 1, N, d)
    k[0, 0, 5800, 5] = np.inf
    row0 = 5760
    assert plan_of(variant, 1, 4, 2, 1, row0, N, d, True)[1] > 1
    o = gpu_attn_chunks(q, k, v, True, scale, [(0, 1, row0)], variant=variant)
    for h in range(4):
        _check(o[0, h], q[0, h], k[0, h // 2], v[0, h // 2], scale, True, variant, row0, 0 if h < 2 else N, "rows")


@pytest.mark.parametrize("variant", [P.MIXED, P.DIRECT])
@pytest.mark.parametrize("N,inf_key", [(1000, 700), (1000, 127), (1000, 999)])
def test_infinite_key_many_rows_d64(N, inf_key, variant):
    rng = np.random.default_rng(N + inf_key)
    B, H, d, scale = 14, 6, 64, f32(0.125)
    q, k, v = _inputs(rng, B, H, H, N, N, d)
    k[3, 2, inf_key, 5] = np.inf
    assert plan_of(variant, B, H, H, N, 0, N, d, True) == ("fwd4", 1)
    o, _ = gpu_attn(q, k, v, True, scale, variant)
    _check(o[3, 2], q[3, 2], k[3, 2], v[3, 2], scale, True, variant, 0, inf_key // 128 * 128, "fwd4")
    assert np.isfinite(np.delete(o.reshape(B * H, N, d), 3 * H + 2, 0)).all()


@pytest.mark.parametrize("variant", [P.MIXED, P.DIRECT])
def test_infinite_key_many_rows_d64_keys_in_pieces(variant):
    rng = np.random.default_rng(77)
    N, d, scale = 9000, 64, f32(0.125)
    q, k, v = _inputs(rng, 1, 2, 2, N, N, d)
    k[0, 1, 8100, 5] = np.inf
    assert plan_of(variant, 1, 2, 2, N, 0, N, d, True)[0] == "fwd4" and plan_of(variant, 1, 2, 2, N, 0, N, d, True)[1] > 1
    o, _ = gpu_attn(q, k, v, True, scale, variant)
    lo = 8000
    _check(o[0, 1, lo:], q[0, 1, lo:], k[0, 1], v[0, 1], scale, True, variant, lo, 8100 // 128 * 128, "fwd4")
    assert np.isfinite(o[0, 0]).all() and np.isfinite(o[0, 1, :lo]).all()


@pytest.mark.parametrize("variant", [P.MIXED, P.DIRECT, P.S16])
@pytest.mark.parametrize("inf_key", [1000, 150, 20])
def test_infinite_key_two_halves(inf_key, variant):
    rng = np.random.default_rng(inf_key)
    N, d, scale = 1100, 128, f32(128 ** -0.5)
    q, k, v = _inputs(rng, 1, 28, 4, N, N, d)
    k[0, 1, inf_key, 5] = np.inf
    assert plan_of(variant, 1, 28, 4, N, 0, N, d, True) == ("halves", 1)
    o, _ = gpu_attn(q, k, v, True, scale, variant)
    _check(o[0, 9], q[0, 9], k[0, 1], v[0, 1], scale, True, variant, 0, inf_key // 128 * 128, "halves")
    assert np.isfinite(np.delete(o[0], slice(7, 14), 0)).all()


@pytest.mark.parametrize("variant", [P.MIXED, P.DIRECT, P.S16])
@pytest.mark.parametrize("B,Hq,Hkv,N,d,inf_key,kernel", [
    (1, 28, 4, 2100, 128, 1990, "halves"), (1, 28, 4, 2100, 128, 150, "halves"),           # with MFMAs of 16 rows
    (1, 28, 4, 3000, 128, 2900, "fwd"), (1, 28, 4, 3000, 128, 300, "fwd"),
    (14, 6, 6, 2500, 64, 2400, "fwd4"),                                                    # on the tiles whose P is made without the maximum
])
def test_infinite_key_longer_sequences(B, Hq, Hkv, N, d, inf_key, kernel, variant):
    rng = np.random.default_rng(N + inf_key)
    scale, G = f32(d ** -0.5), Hq // Hkv
    q, k, v = _inputs(rng, B, Hq, Hkv, N, N, d)
    k[0, 1, inf_key, 5] = np.inf
    if variant != P.S16:
        assert plan_of(variant, B, Hq, Hkv, N, 0, N, d, True) == (kernel, 1)
    o, _ = gpu_attn(q, k, v, True, scale, variant)
    for at in (slice(0, 400), slice(N - 500, N)):
        _check(o[0, G, at], q[0, G, at], k[0, 1], v[0, 1], scale, True, variant, at.start, inf_key // 128 * 128, kernel)
    assert np.isfinite(np.delete(o[0], slice(G, 2 * G), 0)).all() and np.isfinite(o[1:]).all()


def test_bf16_key_beyond_the_fp16_range():
    rng = np.random.default_rng(3)
    N, d, scale = 256, 128, f32(128 ** -0.5)
    q, k, v = (po.fl(rng.standard_normal((1, 1, N, d)), "bf16").astype(np.float32) for _ in range(3))
    k[0, 0, 200, 7] = 131072.0
    assert plan_of(P.MIXED, 1, 1, 1, N, 0, N, d, True) == ("rows", 1)
    o, _ = gpu_attn(q, k, v, True, scale, P.MIXED, bf16=True)
    assert np.isnan(o[0, 0, 128:]).all() and np.isfinite(o[0, 0, :128]).all()


# ------------------------------------------------------------------ S16: finite inputs, one score beyond the fp16 range

def _overflowing(rng, Hq, Hkv, Nq, N, d, at, sign=-1.0):
    """S' of key `at` is about sign * 1e5 for every row; the other keys of its tile move by less than 1000."""
    q, k, v = _inputs(rng, 1, Hq, Hkv, Nq, N, d)
    q[..., 5] = 40.0
    k[0, :, at, 5] = sign * 1e5 / (40.0 * f32(d ** -0.5))
    return q, k, v


@pytest.mark.parametrize("sign", [-1.0, 1.0])
@pytest.mark.parametrize("d,N,at", [(128, 300, 70), (64, 300, 200), (128, 100, 30), (64, 650, 600), (128, 65, 64)])
def test_overflowing_score_few_rows(d, N, at, sign):
    rng = np.random.default_rng(N + at)
    q, k, v = _overflowing(rng, 2, 2, N, N, d, at, sign)
    scale = f32(d ** -0.5)
    assert plan_of(P.S16, 1, 2, 2, N, 0, N, d, True) == ("rows", 1)
    o, _ = gpu_attn(q, k, v, True, scale, P.S16)
    # rows of the first tile: -inf is a weight of zero, +inf is NaN for the rows that see the key
    first = max(at // 128 * 128, 128) if sign < 0 else at if at < 128 else at // 128 * 128
    for h in range(2):
        _check(o[0, h], q[0, h], k[0, h], v[0, h], scale, True, P.S16, 0, first, "rows", at // 128 * 128)


@pytest.mark.parametrize("at", [100, 3333, 5999])
def test_overflowing_score_decoding_step(at):
    rng = np.random.default_rng(at)
    N, d, scale = 6000, 128, f32(128 ** -0.5)
    q, k, v = _overflowing(rng, 4, 2, 3, N, d, at)
    assert plan_of(P.S16, 1, 4, 2, 3, N - 3, N, d, True)[1] > 1
    o = gpu_attn_chunks(q, k, v, True, scale, [(0, 3, N - 3)], variant=P.S16)
    for h in range(4):
        _check(o[0, h], q[0, h], k[0, h // 2], v[0, h // 2], scale, True, P.S16, N - 3, 0, "rows")


@pytest.mark.parametrize("N,at", [(1100, 30), (1100, 150), (1100, 300), (1100, 1050), (1024, 1000)])
def test_overflowing_score_two_halves(N, at):
    rng = np.random.default_rng(N + at)
    d, scale = 128, f32(128 ** -0.5)
    q, k, v = _overflowing(rng, 28, 4, N, N, d, at)
    assert plan_of(P.S16, 1, 28, 4, N, 0, N, d, True) == ("halves", 1)
    o, _ = gpu_attn(q, k, v, True, scale, P.S16)
    for h in (0, 27):
        _check(o[0, h], q[0, h], k[0, h // 7], v[0, h // 7], scale, True, P.S16, 0, max(at // 128 * 128, 128), "halves", at // 128 * 128)


@pytest.mark.parametrize("at", [2100, 2000, 5])
def test_overflowing_score_where_a_range_of_the_key_split_is_one_tile(at):
    """17 key tiles in two ranges, the second of a single tile; with a counter, so that 256-row workgroups take it."""
    import torch
    rng = np.random.default_rng(at)
    N, Nq, d, scale, dev = 2176, 32, 128, f32(128 ** -0.5), torch.device("cuda:0")
    q, k, v = _overflowing(rng, 2, 1, Nq, N, d, at)
    assert plan_of(P.S16, 1, 2, 1, Nq, 0, N, d, False, counters=True) == ("fwd", 2)
    tq, tk, tv = (torch.from_numpy(x).to(dev) for x in (q, k, v))
    wsb = P.pasa_attn_fwd_workspace(1, 2, 1, N, d)
    ws, to = torch.empty(wsb, dtype=torch.uint8, device=dev), torch.zeros_like(tq)
    cnt = torch.zeros(2, dtype=torch.int64, device=dev)
    P.pasa_prepare_kv(tk, tv, 1, 1, N, d, scale, ws, wsb, variant=P.S16)
    P.pasa_attn_fwd_chunk(tq, to, 1, 2, 1, Nq, 0, N, d, False, scale, ws, wsb, variant=P.S16, overflow_s=cnt[0:1], nonfinite_o=cnt[1:2])
    torch.cuda.synchronize()
    assert np.isnan(po.pasa_rows(q[0, 0], k[0, 0], v[0, 0], scale, False, BETA, 128, po.PARTIAL16)).all()
    assert torch.isnan(to).all() and cnt.tolist() == [2 * Nq, 2 * Nq * d]
