"""The calls that a user of this library makes, as cases to be timed and compared.

Four kinds of work, each through its public entry point:

  prompt   one pass over whole sequences: pasa_attn_fwd_ex with a workspace that the caller keeps, or pasa_attn_fwd,
           which brings its own
  chunk    query rows against keys and values that pasa_prepare_kv has laid out before: a decoding step (a few rows
           at the end of a sequence), a piece of a long prompt, cross-attention
  cache    keys and values laid out and the first row attended to: what a server does when a prompt's keys arrive
           from elsewhere

The sizes are those of the five workloads of `workloads/` (one head with d = 64, eight heads with a large key bias, 28
query heads on 4 KV heads with d = 128, 14 x 5 heads with d = 64, the same 28 heads at 32768 keys), the sequence lengths
in between, and the ragged lengths that prompts and caches really have.  The values are drawn like those workloads'.
"""
import math

import torch

import paper_2503_01873_amd as P

VARIANT = {"mixed": P.MIXED, "strict16": P.STRICT16, "s16": P.S16, "direct": P.DIRECT}


def _case(name, work, B, Hq, Hkv, N, d, causal, values, Nq=0, variant="mixed", dtype="f16", entry="ex"):
    return {"name": name, "work": work, "B": B, "Hq": Hq, "Hkv": Hkv, "N": N, "Nq": Nq or N, "d": d, "causal": causal,
            "values": values, "variant": variant, "dtype": dtype, "entry": entry}


def listed():
    return [
        # the smallest call: one head of 256 rows; launches and host work are all there is
        _case("one_head_256", "prompt", 1, 1, 1, 256, 64, False, "bias4"),
        # a chat turn of no round length, in the type that models are stored in
        _case("prompt_777_bf16", "prompt", 1, 28, 4, 777, 128, True, "normal", dtype="bf16"),
        # an ordinary prompt through the simplest entry point, which brings its own workspace
        _case("prompt_2048_plain", "prompt", 1, 28, 4, 2048, 128, True, "outliers", entry="plain"),
        # eight heads without grouping, not causal, keys with the large bias that overflows an unshifted fp16 score
        _case("bias_4096", "prompt", 1, 8, 8, 4096, 128, False, "bias80"),
        # the benchmark's prompt
        _case("prompt_8192", "prompt", 1, 28, 4, 8192, 128, True, "outliers"),
        # spatial attention over the frames of a video: d = 64, many heads, not causal
        _case("frames_9216_d64", "prompt", 14, 5, 5, 9216, 64, False, "resonance"),
        # a long prompt, two sequences
        _case("long_32768_b2", "prompt", 2, 28, 4, 32768, 128, True, "blocks"),
        # Algorithm 1 as printed (every quantity in fp16), a prompt of ragged length
        _case("strict16_4001", "prompt", 1, 28, 4, 4001, 128, True, "normal", variant="strict16"),
        # a decoding step of one long sequence
        _case("decode_32768", "chunk", 1, 28, 4, 32768, 128, True, "blocks", Nq=1),
        # a decoding step of sixteen sequences of a ragged length
        _case("decode_b16_4999", "chunk", 16, 28, 4, 4999, 128, True, "normal", Nq=1),
        # a piece of a long prompt against what is already there
        _case("piece_512_of_16384", "chunk", 1, 28, 4, 16384, 128, True, "outliers", Nq=512),
        # keys of eight prompts laid out, and the first row
        _case("cache_b8_8192", "cache", 8, 28, 4, 8192, 128, True, "normal", Nq=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_LARGEST = 4.0 * 2 * 28 * 32768.0 ** 2 * 128 / 2


def draw(rng):
    while True:
        work = rng.choice(["prompt", "prompt", "prompt", "chunk", "chunk", "cache"])
        Hq, Hkv, d = rng.choice([(1, 1, 64), (8, 8, 128), (28, 4, 128), (28, 4, 128), (28, 4, 128), (5, 5, 64), (12, 2, 128),
                                 (16, 16, 64), (32, 8, 128)])
        B = rng.choice([1, 1, 1, 2, 4, 14])
        N = _log(rng, 128, 32768)
        if rng.random() < 0.4:
            N = max(128, N // 128 * 128)
        causal = rng.random() < 0.7
        values = rng.choice(["normal", "bias4", "outliers", "blocks"] if d == 128 else ["normal", "bias4", "resonance"])
        variant, dtype, entry, Nq = rng.choice(["mixed"] * 5 + ["direct", "strict16", "s16"]), "f16", "ex", N
        if rng.random() < 0.25:
            dtype = "bf16"
        if work == "prompt":
            if variant == "mixed" and dtype == "f16" and rng.random() < 0.25:
                entry = "plain"
        elif work == "chunk":
            # decoding steps, a few proposed tokens, pieces of a prompt
            Nq = rng.choice([1, 1, 2, 5, 8, _log(rng, 16, 2048)])
            Nq = min(Nq, N)
        else:
            Nq = 1
        if variant in ("strict16", "s16"):
            values = "normal"
        c = _case("", work, B, Hq, Hkv, N, d, causal, values, Nq, variant, dtype, entry)
        del c["name"]
        if work_flops(c) <= _LARGEST and B * (Hq * Nq + 4 * Hkv * N) * d <= 1 << 29:
            return c


def _scale(c):
    return float(torch.tensor(c["d"] ** -0.5, dtype=torch.float32))


def _inputs(c, seed):
    """q, k, v on the GPU, drawn like the values of the library's own workloads."""
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(1000003 * int(seed) + 17)
    dt = torch.float16 if c["dtype"] == "f16" else torch.bfloat16
    B, Hq, Hkv, N, Nq, d = (c[x] for x in ("B", "Hq", "Hkv", "N", "Nq", "d"))

    def normal(*shape):
        return torch.randn(shape, generator=g, device=dev, dtype=torch.float32)

    q, k, v = normal(B, Hq, Nq, d), normal(B, Hkv, N, d), normal(B, Hkv, N, d).to(dt)
    kind = c["values"]
    if kind == "bias4":                 # a constant key bias
        k += 4.0
    elif kind == "bias80":              # the unscaled product averages 81920, beyond fp16
        q += 8.0
        k = 80.0 + 2.0 * k
    elif kind == "outliers":            # four channels per KV head: queries 20 times as large, keys + 60
        for b in range(B):
            for h in range(Hkv):
                ch = torch.randperm(d, generator=g, device=dev)[:4]
                q[b, h * (Hq // Hkv):(h + 1) * (Hq // Hkv)][..., ch] *= 20.0
                k[b, h][..., ch] += 60.0
    elif kind == "resonance":           # queries and keys share a wave along the channels, in phase or in antiphase
        phase = 2 * math.pi * torch.rand((B, Hkv, 1, 1), generator=g, device=dev)
        wave = 2 * math.pi * 4.0 * torch.arange(d, device=dev) / d
        anti = math.pi * (torch.arange(Hkv, device=dev) % 2).view(1, Hkv, 1, 1)
        q += 30.0 * torch.sin(wave + phase).repeat_interleave(Hq // Hkv, 1)
        k += 30.0 * torch.sin(wave + phase + anti)
    elif kind == "blocks":              # a key bias that changes every 1024 keys
        bias = 20.0 + 40.0 * torch.rand((B, Hkv, (N + 1023) // 1024), generator=g, device=dev)
        k += bias.repeat_interleave(1024, 2)[:, :, :N, None]
    return q.to(dt), k.to(dt), v


def _row0(c):
    return c["N"] - c["Nq"] if c["causal"] else 0


def prepare(c, seed):
    q, k, v = _inputs(c, seed)
    B, Hq, Hkv, N, d = (c[x] for x in ("B", "Hq", "Hkv", "N", "d"))
    s = {"c": c, "q": q, "o": torch.empty_like(q), "scale": _scale(c),
         "opts": {"variant": VARIANT[c["variant"]], "io_dtype": P.IO_BF16 if c["dtype"] == "bf16" else P.IO_F16}}
    if c["entry"] == "ex":
        s["bytes"] = P.pasa_attn_fwd_workspace(B, Hq, Hkv, N, d)
        s["ws"] = torch.empty(s["bytes"], dtype=torch.uint8, device=q.device)
    if c["work"] == "chunk":
        P.pasa_prepare_kv(k, v, B, Hkv, N, d, s["scale"], s["ws"], s["bytes"], torch.cuda.current_stream(), **s["opts"])
    else:
        s["k"], s["v"] = k, v
    return s


def run(s):
    c, stream = s["c"], torch.cuda.current_stream()
    B, Hq, Hkv, N, Nq, d, causal = (c[x] for x in ("B", "Hq", "Hkv", "N", "Nq", "d", "causal"))
    if c["work"] == "prompt":
        if c["entry"] == "plain":
            P.pasa_attn_fwd(s["q"], s["k"], s["v"], s["o"], B, Hq, Hkv, N, d, causal, s["scale"], stream)
        else:
            P.pasa_attn_fwd_ex(s["q"], s["k"], s["v"], s["o"], B, Hq, Hkv, N, d, causal, s["scale"], s["ws"], s["bytes"], stream,
                               **s["opts"])
        return s["o"]
    if c["work"] == "cache":
        P.pasa_prepare_kv(s["k"], s["v"], B, Hkv, N, d, s["scale"], s["ws"], s["bytes"], stream, **s["opts"])
    P.pasa_attn_fwd_chunk(s["q"], s["o"], B, Hq, Hkv, Nq, _row0(c), N, d, causal, s["scale"], s["ws"], s["bytes"], stream,
                          **s["opts"])
    return s["o"]


def _pairs(c):
    """(query, key) pairs of one head."""
    N, Nq = c["N"], c["Nq"]
    if not c["causal"]:
        return float(N) * Nq
    return Nq * float(_row0(c)) + Nq * (Nq + 1) / 2.0


def work_flops(c):
    return 4.0 * c["d"] * c["B"] * c["Hq"] * _pairs(c)


def work(c):
    rows, keys = c["B"] * c["Hq"] * c["Nq"] * c["d"], c["B"] * c["Hkv"] * c["N"] * c["d"]
    moved = 2 * 2 * rows + 2 * 2 * keys          # q and o, k and v (or what was laid out from them)
    if c["work"] == "cache":
        moved += 2 * 2 * keys                    # what is laid out stays for the rows to come
    return {"bytes": moved, "flops": work_flops(c)}


# What the order of the sums and the reference level of P leave open: P is rounded to fp16 once, relative to whatever level
# its row's output is stored at, and the output to its own type.  Measured as the 2-norm between two runs of the same
# case, once with the channels (and, where nothing is masked, the keys of a tile) in another order, which moves only the
# rounding of fp32 sums (up to 1.8e-4; fp16 statistics 6.1e-4; bf16 outputs 4.0e-4), and once with the keys of a row
# swept in other pieces, which moves the levels too (3.7e-4).  Four times that is 1.5e-3 to 2.4e-3; single values differed by up
# to 5.8e-3 (fp16) and by one step, 7.8e-3 (bf16).
def tolerance(c):
    if c["dtype"] == "bf16":
        return {"rel": 4e-3, "max": 0.04}
    return {"rel": 2.4e-3 if c["variant"] == "strict16" else 2e-3, "max": 0.03}


def exact(c, seed):
    """softmax(scale * q k^T) v in 64 bits, rows in pieces."""
    q, k, v = _inputs(c, seed)
    B, Hq, Hkv, N, Nq = (c[x] for x in ("B", "Hq", "Hkv", "N", "Nq"))
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    pos = torch.arange(Nq, device=q.device) + _row0(c)
    step = max(1, (1 << 26) // N)
    for b in range(B):
        for h in range(Hkv):
            kt, vd = k[b, h].double().t().contiguous(), v[b, h].double()
            for hq in range(h * (Hq // Hkv), (h + 1) * (Hq // Hkv)):
                for r in range(0, Nq, step):
                    e = min(Nq, r + step)
                    n = min(N, _row0(c) + e) if c["causal"] else N
                    s = (q[b, hq, r:e].double() @ kt[:, :n]) * _scale(c)
                    if c["causal"]:
                        s.masked_fill_(torch.arange(n, device=q.device)[None, :] > pos[r:e, None], -math.inf)
                    s -= s.amax(1, keepdim=True)
                    s.exp_()
                    out[b, hq, r:e] = (s @ vd[:n]) / s.sum(1, keepdim=True)
    return out
