// PASA attention for few query rows (decoding steps, proposed tokens, short prompts): pasa_rows, and the merge of key
// splits that it shares with pasa_fwd.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "pasa_device.h"
#include "pasa_kernels.h"

namespace {

constexpr int U = 64;           // keys per unit of work of one wavefront (half a tile)
constexpr float CMAX = 8.f;     // P may exceed 1 by at most e^CMAX before a row moves its stored output to a new level
constexpr float PMAX = 2980.f;  // the fp16 value below e^CMAX

__device__ inline h8 load_frag(__amdgpu_buffer_rsrc_t src, int voff, int soff)
{
    return __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(src, voff, soff, 0));
}

// One workgroup = NW wavefronts owns 16 * RB rows and a range of the keys in units of 64.  The rows come from lists: with fewer than 16 rows given, the rows of ALL the
// heads that share a KV head are one list (they are contiguous in q and o), so that a decoding step reads its keys once;
// otherwise each head is a list, so that a block's rows are neighbours in position.  Every wavefront sweeps units of its
// own for all of the rows and the wavefronts' states are merged through LDS at the end: no key or value is read twice
// by a workgroup, no wavefront waits for another before the end, and nothing has to be staged: the workspace is laid
// out in fragments, which go from memory straight to the registers that the matrix cores read.
//
// GEMMs on v_mfma_f32_16x16x32_f16, transposed like pasa_fwd's: S'^T = K' Q^T and O^T += V^T P^T.  Lane l holds query row
// l % 16, and with g = l / 16 the four keys 4g .. 4g+3 of a 16-key block.  Which keys a block consists of is free: block
// 2i + s of a unit takes keys 32i + {0..7, 16..23} + 8s, which makes the P of blocks 2i and 2i + 1 the B operand of one
// k-step whose A operand is one 16-byte chunk of the V tile.
//
// The level of a row's stored output is kept as one number R (fp64): the scores of a tile stand for S' + bias, with bias =
// inva * Sbar' (MIXED: what the two correction terms of Algorithm 1's step 3 add up to, m + inva * F + Lc; F cancels)
// or scale * (q . k0) (DIRECT).
//
// What bounds it: a few rows, the keys' way from memory (one row of 32768 keys, 28 heads on 4: 67 MB, 15 us; a large read
// reaches 6 TB/s here); more rows, the vector memory path into the registers (36 KB for a unit and wavefront, 46 bytes a
// clock and compute unit in 128 rows of 32768 keys, 147 us), which is why 32 rows take hardly longer than 16.  So a lane's
// work per score is kept to a multiply-add, an exponential and half a pack: row sums come from the matrix core (P against
// ones), the pseudo-average needs no exchange (the even rows of its A operand are the high parts of the tile's mean, the
// odd rows the low parts), and the level is kept in absolute terms.  (With row sums in lanes and the products for eight
// tiles at a time shared out by shuffles, 32 rows took twice as long as 16.)  Four wavefronts per workgroup: two workgroups
// share a compute unit, so that one loads while the other merges (28 heads of 512 rows 16.8 -> 11.7 us against eight).
template <int D, int RB, int NW, bool S16>
__global__ __launch_bounds__(64 * NW, 2)
void pasa_rows(const _Float16* __restrict__ q, const char* __restrict__ ws, const _Float16* __restrict__ kmean,
               _Float16* __restrict__ o, FastDiv lists, FastDiv Nq_, FastDiv nblk_, FastDiv nsplit_, int grid, int list_rows, int row0, int N,
               int causal, int units, float coef, int mixed, int io_bf16, const unsigned long long* gate,
               float* __restrict__ part_o, double* __restrict__ part_lr, size_t rows_all)
{
    constexpr int KS = D / 32;                   // k-steps of the first GEMM
    constexpr int CB = D / 16;                   // 16-channel blocks of O^T
    constexpr int ROWS = 16 * RB;
    constexpr int LD = D + 4;                    // LDS row of the merge, in floats
    constexpr int TILE_BYTES = 4 * T * D;        // K' tile then V tile
    // S16, d = 64: P without the maximum of its scores, as in pasa_fwd (14 x 5 heads of 366 rows 22.7 -> 21.5 us).  Not MIXED: 4 heads, 700 rows of 12800
    // keys 29.3 -> 28.6 us with normal values, but 29.5 -> 32.3 where rows keep rising and P is made twice (resonant values).  d = 128 waits
    // for its fragments, not for this chain (128 rows of 20000 keys 91.4 / 91.0), and with 32 rows has no registers to keep the scores beside P.
    constexpr bool LEVEL = D == 64 && S16;
    __shared__ __attribute__((aligned(16))) float lds_o[NW * ROWS * LD];
    __shared__ double lds_r[NW][ROWS];
    __shared__ float lds_l[NW][ROWS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 15, g = lane >> 4;

    // Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its own: every XCD gets a contiguous range of the
    // work, in which the row blocks that read the same keys follow one another.  14 x 28 heads on 4, 64 rows of
    // 6000 keys: 124 us; with neighbours on different XCDs, where every L2 fetches every key, 241 us
    // Not for a single causal list, whose last range is the longest (one head of 16384 rows 173 -> 123 us).
    const int Nq = (int)Nq_.d, nblk = (int)nblk_.d, nsplit = (int)nsplit_.d;
    unsigned idx = blockIdx.x;
    if (!causal || row0 >= Nq || grid != nblk * nsplit) {
        const unsigned x = idx & 7, whole = (unsigned)grid >> 3, rest = grid & 7;
        idx = x * whole + (x < rest ? x : rest) + (idx >> 3);
    }
    // causal: the longest blocks of a list first (8 heads of 3000 rows 38.0 -> 36.6 us, 5 of 8000 92.6 -> 86.4); not where a
    // block has four units per wavefront at most (28 heads of 777 rows 19.6 us, longest first 21.1; of 1024 rows 25.7 / 25.1)
    unsigned up = nblk_.quotient(idx);
    int blk = (int)nblk_.rest(idx, up);
    if (causal && N > 1024) blk = nblk - 1 - blk;
    idx = up;
    up = lists.quotient(idx);
    const int list = (int)lists.rest(idx, up);
    const unsigned kv_group = nsplit_.quotient(up);
    const int split = (int)nsplit_.rest(up, kv_group);
    const size_t grp = kv_group;                 // b * Hkv + hk
    if (gate != nullptr && gate[grp] == 0) return;   // adaptive start: nothing overflowed here
    const size_t list0 = (grp * lists.d + list) * (size_t)list_rows;   // first row of the list, in q and o
    const int p0 = blk * ROWS;
    int p1 = p0 + ROWS - 1;
    if (p1 > list_rows - 1) p1 = list_rows - 1;

    // keys seen by the block's rows: all up to the last position (causal), from the first position on only in part
    const int h0 = (int)Nq_.quotient(p0), h1 = (int)Nq_.quotient(p1);
    int first_pos = N - 1, last_pos = N - 1;
    if (causal) {
        const int lo = row0 + (h0 == h1 ? p0 - h0 * Nq : 0), hi = row0 + (h0 == h1 ? p1 - h1 * Nq : Nq - 1);
        if (lo < first_pos) first_pos = lo;
        if (hi < last_pos) last_pos = hi;
    }
    const int U_blk = last_pos / U + 1;                          // units the block needs
    const int us = split * units;                                // this workgroup's: [us, ue)
    int ue = us + units;
    if (ue > U_blk) ue = U_blk;
    // dealt out one by one: without a key split a row's result does not depend on the rows it shares a workgroup with
    const int u0 = us + wave;

    const int ntile = (N + T - 1) / T, nblk16 = (ntile + 15) >> 4;
    const __amdgpu_buffer_rsrc_t tiles = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(ws) + grp * (size_t)ntile * TILE_BYTES, 0, ntile * TILE_BYTES, 0x00020000);
    const __amdgpu_buffer_rsrc_t means = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<_Float16*>(kmean) + grp * (size_t)nblk16 * (32 * D), 0, nblk16 * 64 * D, 0x00020000);

    // lane offsets of the fragments
    const int kv = (g * T + 16 * (lq >> 3) + (lq & 7)) * 16;     // row r of a block is key 16 (r / 8) + r % 8 of its 32: see kfrag
    const int vv = ((g >> 1) * 2 * D + (g & 1) * D + lq) * 16;
    const int mv = (g * 32 + 4 * (lq & 1)) * 16;                 // rows 8 (t / 4) + t % 4 (high) and 4 further down (low)

    // Three register buffers of half a unit's keys or values (8 KB each at d = 128) take the four halves in turn: A holds K' of
    // the first half of the channels, then V of the second half of the keys; B K' of the other channels; C V of the other keys.
    // Each is loaded again as soon as the products with it are done.
    constexpr int HF = CB;                                       // fragments of a half
    h8 A[HF], B[HF], C[HF];
    auto load_k = [&](h8 (&dst)[HF], int u, int half) {
        const int base = (u >> 1) * TILE_BYTES + (u & 1) * (U * 16) + half * (KS / 2) * (4 * T * 16);
#pragma unroll
        for (int n = 0; n < HF; ++n)                             // block n % 4, k-step n / 4 of the half
            dst[n] = load_frag(tiles, kv, base + (n / 4) * (4 * T * 16) + ((n % 4) >> 1) * (32 * 16) + (n & 1) * (8 * 16));
    };
    h8 Am[KS];                                                   // even rows: high, odd rows: low part of the tile's mean
    auto load_m = [&](int u) {
        const int t = u >> 1;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            Am[ks] = load_frag(means, mv, (t >> 4) * (64 * D) + ((t & 12) * 2 + (t & 3)) * 16 + ks * (4 * 32 * 16));
    };
    auto load_v = [&](h8 (&dst)[HF], int u, int half) {
        const int base = (u >> 1) * TILE_BYTES + 2 * T * D + (u & 1) * (U * 2 * D) + half * (4 * D * 16);
#pragma unroll
        for (int n = 0; n < HF; ++n) dst[n] = load_frag(tiles, vv, base + n * (16 * 16));   // channel block n
    };

    constexpr bool QLDS = RB > 1;                // the query fragments wait in LDS: the registers are needed for RB * 2 blocks
    __shared__ __attribute__((aligned(16))) h8 lds_q[QLDS ? RB * KS * 64 : 1];
    h8 Qr[QLDS ? 1 : RB][KS];
    auto Qf = [&](int rb, int ks) { return QLDS ? lds_q[(rb * KS + ks) * 64 + lane] : Qr[QLDS ? 0 : rb][ks]; };
    f4 O[RB][CB];
    f4 L[RB];                                    // row sums of P, the same in all elements
    double R[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        L[rb] = (f4)0.f;
        R[rb] = -__builtin_inf();
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) O[rb][cb] = (f4)0.f;
    }

    // Query rows first: loads come back in the order they were asked for, and nothing can begin without these (behind the first keys
    // and values they took 2.0 us of a workgroup's 8.9 in 28 heads of 777 rows).  Rows past the
    // list's end are out of the buffer's bounds and come as zeros.  The buffer is the block's, not the list's: a list may be longer than
    // the 4 GiB that a buffer's size and offsets count.
    const __amdgpu_buffer_rsrc_t rows_in =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(q + (list0 + p0) * D), 0, (p1 + 1 - p0) * (2 * D), 0x00020000);
    constexpr int QN = QLDS ? RB * KS / NW : RB * KS;            // fragments that this wavefront loads: to be shared, or all of its own
    h8 raw[QN];
#pragma unroll
    for (int n = 0; n < QN; ++n) {
        const int at = QLDS ? n * NW + wave : n;                 // fragment: row block at / KS, k-step at % KS
        raw[n] = load_frag(rows_in, lq * (2 * D) + 16 * g + at / KS * (32 * D), 64 * (at % KS));
    }
    PASA_FENCE();
    // the half tile whose keys A and B take first for unit u
    auto first_k = [](int u) { return S16 ? u ^ 1 : u; };
    if (u0 < ue) {
        if (!S16) load_m(u0);
        load_k(B, first_k(u0), 1);
        load_k(A, first_k(u0), 0);
        load_v(C, u0, 0);
        if (!QLDS) PASA_FENCE();
    }
    if (QLDS) PASA_FENCE();
    int last[RB];                                // last key that the lane's row sees
    auto take_rows = [&] {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int p = p0 + 16 * rb + lq;
            last[rb] = N - 1;
            if (causal && p < list_rows) {
                const int pos = row0 + (int)Nq_.rest(p, Nq_.quotient(p));
                if (pos < N - 1) last[rb] = pos;
            }
        }
        if (io_bf16) {
#pragma unroll
            for (int n = 0; n < QN; ++n) raw[n] = bf16x8_to_h8(__builtin_bit_cast(u16x8, raw[n]));
        }
#pragma unroll
        for (int n = 0; n < QN; ++n) {
            if (QLDS) lds_q[(n * NW + wave) * 64 + lane] = raw[n];
            else Qr[QLDS ? 0 : n / KS][n % KS] = raw[n];
        }
    };
    if (QLDS) {
        take_rows();
        __syncthreads();
    }
    // Rows that stay in registers are taken on the way that has keys to sweep, behind its loads: where the ways with and without meet,
    // the compiler has to take the rows for the newest loads, and then its wait, at their first use in the loop, is for all the
    // keys on their way, in every iteration (16 heads, d = 64, 128 rows of 28000 keys 88.7 us, so 80.1; d = 128, 28 heads on 4, 64 rows of
    // 20000 keys 92.3 / 89.1).
    if (u0 < ue) {
        if (!QLDS) take_rows();
        // d = 64: the four wavefronts start a quarter of an iteration apart (1300 clocks, of which their fragments keep the first-level
        // cache busy for 1150).  In step, all load and all compute at the same time, and they stay in step: workgroups of one launch
        // took 27 us or 34.  4 heads, 700 rows of 12800 keys 35.9 -> 29.4 us.  Not for a few iterations (no difference up to four), nor
        // where arithmetic keeps them apart: d = 128 (28 heads on 4, 128 rows of 20000 keys 91.2 -> 94.9), fp16 scores (103.0 -> 105).
        if (!QLDS && !S16 && D == 64 && ue - us > 4 * NW)
            for (int i = 0; i < wave; ++i) __builtin_amdgcn_s_sleep(5);      // 320 clocks each
        auto unit = [&](int u, auto more_c) {
            constexpr bool more = decltype(more_c)::value;
            const int t = u >> 1;
            // q . mean of the tile: every lane gets the product with the high part in element 0, with the low part in 1
            f4 M[RB];
            if (!S16) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) M[rb] = (f4)0.f;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        M[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(Am[ks], Qf(rb, ks), M[rb], 0, 0, 0);
                PASA_FENCE();
                if (more) load_m(u + NW);
            }
            f4 S[RB][4];
            auto gemm1 = [&](const h8 (&k)[HF], int half, bool clear) {
#pragma unroll
                for (int ks = 0; ks < KS / 2; ++ks) {
                    h8 qf[RB];
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) qf[rb] = Qf(rb, half * (KS / 2) + ks);
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb)
                            S[rb][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(k[4 * ks + b], qf[rb], clear && ks == 0 ? (f4)0.f : S[rb][b], 0, 0, 0);
                }
                PASA_FENCE();
            };
            PASA_FENCE();
            // S16: the pseudo-average is the mean of the tile's rounded scores, those of its other half included
            float sum[RB];
            auto round_and_add = [&](bool other) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    float x = 0.f;
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            S[rb][b][i] = (float)(_Float16)S[rb][b][i];
                            x += S[rb][b][i];
                        }
                    sum[rb] = other ? x : sum[rb] + x;
                }
            };
            if (S16) {
                gemm1(B, 1, true);
                load_k(B, u, 1);
                PASA_FENCE();
                gemm1(A, 0, false);
                load_k(A, u, 0);
                PASA_FENCE();
                round_and_add(true);
            }
            gemm1(B, 1, true);
            if (more) load_k(B, first_k(u + NW), 1);
            PASA_FENCE();
            gemm1(A, 0, false);
            load_v(A, u, 1);
            PASA_FENCE();
            if (S16) round_and_add(false);

            const int tail = N - t * T;          // keys of this tile, when fewer than 128
            h8 P[RB][2];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if (rb > 0) PASA_FENCE();
                float v;
                if (S16) {
                    v = sum_row(sum[rb]) * (tail < T ? 1.0f / (float)tail : 1.0f / T);
                } else {
                    v = M[rb][0] + M[rb][1] * 0.00048828125f;    // low parts are stored times 2^11
                    if (mixed && tail < T) v *= (float)T * (1.0f / (float)tail);
                }
                if (u * U + U - 1 > first_pos) {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (u * U + 32 * (b >> 1) + 16 * (g >> 1) + 8 * (b & 1) + 4 * (g & 1) + i > last[rb]) S[rb][b][i] = -__builtin_inff();
                }
                // A row that sees a single tile needs no bias, which may be infinite: a score that overflowed to -inf only takes
                // its own weight there.
                const bool one_tile = last[rb] < T;
                if (one_tile) v = 0.f;
                const bool seen = last[rb] >= u * U;
                float nml;
                auto exponentials = [&] {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int i = 0; i < 4; i += 2) {
                            const f2 e = {__builtin_amdgcn_exp2f(__builtin_fmaf(S[rb][b][i], LOG2E, nml)),
                                          __builtin_amdgcn_exp2f(__builtin_fmaf(S[rb][b][i + 1], LOG2E, nml))};
                            const h2 ph = __builtin_convertvector(e, h2);
                            P[rb][b >> 1][4 * (b & 1) + i] = ph[0];
                            P[rb][b >> 1][4 * (b & 1) + i + 1] = ph[1];
                        }
                };
                // Rows that `rises` holds for move their stored output to the level of this unit's maximum.  Not "no score above -inf"
                // for a row without keys here: those of keys that it sees may all have overflowed.  c is the unit's level relative to the
                // stored output's (first unit: +inf, which clears the zeros); NaN, and with it the row, where the maximum or the bias is not
                // finite: scores of keys it sees left the range of their type.
                auto move_up = [&](auto rises) {
                    float mx = S[rb][0][0];
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i) mx = __builtin_fmaxf(mx, S[rb][b][i]);
                    mx = max_row(mx);
                    const bool unseen = !seen || (one_tile && mx == -__builtin_inff());
                    const double lev = (double)mx + (double)coef * (double)v;
                    const float bad = (mx + v) * 0.f;
                    float c = (float)(lev - R[rb]) + bad;
                    const bool move = rises(c) && !(LEVEL && unseen);
                    if (__builtin_amdgcn_ballot_w64(move) != 0ull) {
                        const float r = move ? __builtin_amdgcn_exp2f(-c * LOG2E) : 1.f;
                        R[rb] = move ? lev : R[rb];
                        c = move ? bad : c;
                        L[rb] *= r;
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) O[rb][cb] *= r;
                    }
                    if (!LEVEL || move) nml = (c - mx) * LOG2E;
                    if (unseen) nml = 0.f;
                };
                if (!LEVEL) {
                    move_up([](float c) { return c > CMAX; });
                    exponentials();
                } else {
                    nml = 0.f;
                    unsigned long long high = ~0ull;
                    if (__builtin_amdgcn_ballot_w64(R[rb] != -__builtin_inf()) != 0ull) {     // not at the first unit
                        const float off = __builtin_fmaf(v, 0.f, (float)__builtin_fma((double)coef, (double)v, -R[rb]));
                        if (seen) nml = off * LOG2E;
                        exponentials();
                        high = __builtin_amdgcn_ballot_w64(!(largest_of(P[rb]) <= PMAX));
                    }
                    if (high != 0ull) {
                        asm volatile("" ::: "memory");
                        // a row that has risen above its stored output, or has none yet, shows in the P of one of its four lanes
                        const unsigned both = (unsigned)high | (unsigned)(high >> 32);
                        move_up([&](float) { return ((both | both >> 16) >> lq & 1u) != 0u; });
                        exponentials();
                    }
                }
            }
            auto gemm2 = [&](const h8 (&v)[HF], int half) {
#pragma unroll
                for (int n = 0; n < HF; ++n)
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
                        O[rb][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(v[n], P[rb][half], O[rb][n], 0, 0, 0);
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)                  // the row sums of the rounded P
                    L[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16((h8)(_Float16)1, P[rb][half], L[rb], 0, 0, 0);
                PASA_FENCE();
            };
            PASA_FENCE();
            gemm2(C, 0);
            if (more) load_v(C, u + NW, 0);
            PASA_FENCE();
            gemm2(A, 1);
            if (more) load_k(A, first_k(u + NW), 0);
        };
        int u = u0;
        for (; u + NW < ue; u += NW) unit(u, std::true_type{});
        unit(u, std::false_type{});
    }

    // ---- the wavefronts' states brought to the highest of their levels and added ----
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        if (g == 0) lds_r[wave][16 * rb + lq] = R[rb];
    }
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        double rmax = -__builtin_inf();
#pragma unroll
        for (int w = 0; w < NW; ++w) rmax = __builtin_fmax(rmax, lds_r[w][16 * rb + lq]);
        const float wgt = R[rb] == -__builtin_inf() ? 0.f : __builtin_amdgcn_exp2f((float)(R[rb] - rmax) * LOG2E);
        if (g == 0) lds_l[wave][16 * rb + lq] = wgt * L[rb][0];
        float* dst = lds_o + (wave * ROWS + 16 * rb + lq) * LD + 4 * g;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) *reinterpret_cast<f4*>(dst + 16 * cb) = O[rb][cb] * wgt;
    }
    __syncthreads();
    constexpr int STEP = 64 * NW / (D / 8);      // rows that the workgroup writes at a time, eight channels a lane
#pragma unroll
    for (int r0 = 0; r0 < ROWS; r0 += STEP) {
        const int r = r0 + tid / (D / 8), c8 = tid % (D / 8) * 8;
        f4 acc[2] = {(f4)0.f, (f4)0.f};
        float ls = 0.f;
        if (ROWS % STEP != 0 && r >= ROWS) break;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const f4* src = reinterpret_cast<const f4*>(lds_o + (w * ROWS + r) * LD + c8);
            acc[0] += src[0];
            acc[1] += src[1];
            ls += lds_l[w][r];
        }
        const size_t grow = list0 + p0 + r;
        const bool real = p0 + r < list_rows;
        if (nsplit > 1) {
            if (real) {
                f4* dst = reinterpret_cast<f4*>(part_o + ((size_t)split * rows_all + grow) * D + c8);
                dst[0] = acc[0];
                dst[1] = acc[1];
            }
            if (real && c8 == 0) {
                double rmax = -__builtin_inf();
                for (int w = 0; w < NW; ++w) rmax = __builtin_fmax(rmax, lds_r[w][r]);
                part_lr[((size_t)split * rows_all + grow) * 2] = ls;
                part_lr[((size_t)split * rows_all + grow) * 2 + 1] = ls == ls ? rmax : ls;     // NaN stays NaN
            }
        } else {
            const float inv = 1.0f / ls;
            unsigned out[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = acc[e >> 1][2 * (e & 1)] * inv, y = acc[e >> 1][2 * (e & 1) + 1] * inv;
                out[e] = io_bf16 ? pack_bf16(x, y) : pack_f16(x, y);
            }
            if (real) *reinterpret_cast<uint4*>(o + grow * D + c8) = uint4{out[0], out[1], out[2], out[3]};
        }
    }
}

// Merge of the key splits of one call: per query row, the splits' stored outputs and sums are brought to the highest of
// their levels (the log-sum-exp rule on the absolute level a split's stored output refers to: m + Inva * F + Lc in
// pasa_fwd, R in pasa_rows and pasa_fwd4) and added; then Algorithm 1's final quotient.  A split that saw none of a row's keys
// has level -inf and weighs nothing (its output may not be written); NaN stays NaN.
__device__ inline float merge_weight(double level, double top)
{
    return level == -__builtin_inf() ? 0.f : __builtin_amdgcn_exp2f((float)(level - top) * LOG2E);
}

// infinity or NaN, by the bits of the output type: all exponent bits set
__device__ inline unsigned not_finite(unsigned bits, int io_bf16)
{
    const unsigned exponent = io_bf16 ? 0x7f80u : 0x7c00u;
    return (bits & exponent) == exponent ? 1u : 0u;
}

// Many rows: one thread per 8 channels of a row goes through the splits.
template <int D>
__global__ __launch_bounds__(256) void pasa_merge_splits(const float* __restrict__ part_o, const double* __restrict__ part_lr,
                                                         _Float16* __restrict__ o, size_t rows_all, int nsplit, int io_bf16,
                                                         unsigned long long* nonfinite_o)
{
    constexpr int TPR = D / 8;                       // threads per row
    const size_t grow = (size_t)blockIdx.x * (256 / TPR) + threadIdx.x / TPR;
    if (grow >= rows_all) return;
    const int c0 = (threadIdx.x % TPR) * 8;
    double rmax = -__builtin_inf();
    for (int s = 0; s < nsplit; ++s) rmax = __builtin_fmax(rmax, part_lr[((size_t)s * rows_all + grow) * 2 + 1]);
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float lsum = 0.f;
    for (int s = 0; s < nsplit; ++s) {
        const double r = part_lr[((size_t)s * rows_all + grow) * 2 + 1];
        if (r == -__builtin_inf()) continue;
        const float wgt = merge_weight(r, rmax);
        lsum += wgt * (float)part_lr[((size_t)s * rows_all + grow) * 2];
        const f4* src = reinterpret_cast<const f4*>(part_o + ((size_t)s * rows_all + grow) * D + c0);
        const f4 a = src[0], b = src[1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[i] += wgt * a[i];
            acc[4 + i] += wgt * b[i];
        }
    }
    const float inv = 1.0f / lsum;
    unsigned out[4], n_bad = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] *= inv;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        out[e] = io_bf16 ? pack_bf16(acc[2 * e], acc[2 * e + 1]) : pack_f16(acc[2 * e], acc[2 * e + 1]);
        n_bad += not_finite(out[e] & 0xffffu, io_bf16) + not_finite(out[e] >> 16, io_bf16);
    }
    *reinterpret_cast<uint4*>(o + grow * D + c0) = uint4{out[0], out[1], out[2], out[3]};
    if (nonfinite_o != nullptr && n_bad) atomicAdd(nonfinite_o, (unsigned long long)n_bad);
}

// Few rows: one workgroup per row, SL groups of D / 8 threads that take the splits in turn, four at a time with all their
// loads on the way together; bound by the latency of two rounds through memory and LDS (28 rows of 128 splits: 3.7 us; with
// one load after another and a serial sum 6.0).
template <int D, int SL>
__global__ __launch_bounds__(D / 8 * SL) void pasa_merge_row(const float* __restrict__ part_o, const double* __restrict__ part_lr,
                                                             _Float16* __restrict__ o, size_t rows_all, int nsplit, int io_bf16,
                                                             unsigned long long* nonfinite_o)
{
    constexpr int TPR = D / 8;
    __shared__ double lds_r[SL];
    __shared__ float lds_l[SL];
    __shared__ __attribute__((aligned(16))) float lds_o[SL][D];
    const int tid = threadIdx.x, cl = tid % TPR, sl = tid / TPR;
    const size_t row = blockIdx.x;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float l = 0.f;
    double top = -__builtin_inf();                   // of this group's splits so far: what acc and l refer to
    for (int s0 = sl; s0 < nsplit; s0 += 4 * SL) {
        double2 lr[4];
        f4 a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const size_t at = (size_t)(s0 + i * SL < nsplit ? s0 + i * SL : s0) * rows_all + row;
            lr[i] = reinterpret_cast<const double2*>(part_lr)[at];
            const f4* src = reinterpret_cast<const f4*>(part_o + at * D + 8 * cl);
            a[i] = src[0];
            b[i] = src[1];
        }
        double t = top;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (s0 + i * SL < nsplit) t = __builtin_fmax(t, lr[i].y);
        const float keep = merge_weight(top, t);
        l *= keep;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= keep;
        top = t;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (s0 + i * SL >= nsplit || lr[i].y == -__builtin_inf()) continue;
            const float w = merge_weight(lr[i].y, t);
            l += w * (float)lr[i].x;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[e] += w * a[i][e];
                acc[4 + e] += w * b[i][e];
            }
        }
    }
    if (cl == 0) {
        lds_r[sl] = top;
        lds_l[sl] = l;
    }
#pragma unroll
    for (int e = 0; e < 8; e += 4) *reinterpret_cast<f4*>(&lds_o[sl][8 * cl + e]) = f4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
    __syncthreads();
    if (tid >= D) return;
    top = -__builtin_inf();
#pragma unroll
    for (int i = 0; i < SL; ++i) top = __builtin_fmax(top, lds_r[i]);
    float x = 0.f, ls = 0.f;
#pragma unroll
    for (int i = 0; i < SL; ++i) {
        const float w = merge_weight(lds_r[i], top);
        x += w * lds_o[i][tid];
        ls += w * lds_l[i];
    }
    x *= 1.0f / ls;
    const unsigned bits = (io_bf16 ? pack_bf16(x, 0.f) : pack_f16(x, 0.f)) & 0xffffu;
    reinterpret_cast<unsigned short*>(o)[row * D + tid] = (unsigned short)bits;
    if (nonfinite_o != nullptr && not_finite(bits, io_bf16)) atomicAdd(nonfinite_o, 1ull);
}

template <int D>
void launch_merge(const void* part_o, const void* part_lr, void* o, size_t rows_all, int nsplit, int io_bf16,
                  unsigned long long* nonfinite_o, hipStream_t stream)
{
    if (nsplit > 2 && rows_all <= 4096) {
        constexpr int MANY = 32, FEW = 8;
        if (nsplit > 2 * FEW)
            hipLaunchKernelGGL((pasa_merge_row<D, MANY>), dim3((unsigned)rows_all), dim3(D / 8 * MANY), 0, stream, (const float*)part_o,
                               (const double*)part_lr, (_Float16*)o, rows_all, nsplit, io_bf16, nonfinite_o);
        else
            hipLaunchKernelGGL((pasa_merge_row<D, 128 / D * FEW>), dim3((unsigned)rows_all), dim3(128 / 8 * FEW), 0, stream, (const float*)part_o,
                               (const double*)part_lr, (_Float16*)o, rows_all, nsplit, io_bf16, nonfinite_o);
        return;
    }
    constexpr int RPB = 256 / (D / 8);
    hipLaunchKernelGGL(pasa_merge_splits<D>, dim3((unsigned)((rows_all + RPB - 1) / RPB)), dim3(256), 0, stream,
                       (const float*)part_o, (const double*)part_lr, (_Float16*)o, rows_all, nsplit, io_bf16, nonfinite_o);
}

template <int D, int RB, int NW, bool S16 = false>
hipError_t launch_rows(const PasaLaunch& p)
{
    const int G = p.Hq / p.Hkv, lists = p.Nq < 16 ? 1 : G, list_rows = p.Nq < 16 ? G * p.Nq : p.Nq;
    const int nblk = (list_rows + 16 * RB - 1) / (16 * RB);
    const int keys = p.causal && p.row0 < p.N - p.Nq ? p.row0 + p.Nq : p.N;
    const int all = (keys + U - 1) / U, units = (all + p.nsplit - 1) / p.nsplit;
    const int nsplit = (all + units - 1) / units;                 // none without keys
    const size_t rows_all = (size_t)p.B * p.Hq * p.Nq;
    const unsigned grid = (unsigned)((size_t)p.B * p.Hkv * lists * nblk * nsplit);
    auto kern = pasa_rows<D, RB, NW, S16>;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * NW), 0, p.stream,
                       (const _Float16*)p.q, (const char*)p.ws, (const _Float16*)p.kmean, (_Float16*)p.o, fast_div(lists), fast_div(p.Nq),
                       fast_div(nblk), fast_div(nsplit), (int)grid, list_rows, p.row0, p.N, p.causal, units, p.variant == PASA_K_DIRECT ? p.scale : p.inva,
                       p.variant == PASA_K_MIXED ? 1 : 0, p.io_bf16, p.gate, (float*)p.part_o, (double*)p.part_lr, rows_all);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nsplit == 1) return e;
    return pasa_launch_merge(p.part_o, p.part_lr, p.o, rows_all, p.d, nsplit, p.io_bf16, nullptr, p.stream);
}

}  // namespace

hipError_t pasa_launch_merge(const void* part_o, const void* part_lr, void* o, size_t rows_all, int d, int nsplit,
                             int io_bf16, unsigned long long* nonfinite_o, hipStream_t stream)
{
    if (d == 128) launch_merge<128>(part_o, part_lr, o, rows_all, nsplit, io_bf16, nonfinite_o, stream);
    else launch_merge<64>(part_o, part_lr, o, rows_all, nsplit, io_bf16, nonfinite_o, stream);
    return hipGetLastError();
}

hipError_t pasa_launch_rows(const PasaLaunch& p, int row_blocks)
{
    if (p.variant == PASA_K_S16) return p.d == 128 ? launch_rows<128, 1, 4, true>(p) : launch_rows<64, 1, 4, true>(p);
    if (p.d == 128) return row_blocks == 1 ? launch_rows<128, 1, 4>(p) : launch_rows<128, 2, 4>(p);
    return row_blocks == 1 ? launch_rows<64, 1, 4>(p) : launch_rows<64, 2, 4>(p);
}
