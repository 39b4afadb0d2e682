// PASA attention for few query rows (decoding steps, proposed tokens, short prompts): pasa_rows, and the merge of key
// splits that it shares with pasa_fwd.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

#include "pasa_kernels.h"

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int T = 128;          // keys per shift tile
constexpr int U = 64;           // keys per unit of work of one wavefront (half a tile)
constexpr float LOG2E = 1.4426950408889634f;
constexpr float CMAX = 8.f;     // P may exceed 1 by at most e^CMAX before a row moves its stored output to a new level

__device__ inline h8 q_from_bf16(u16x8 raw)
{
    h8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (_Float16)__uint_as_float((unsigned)raw[e] << 16);
    return out;
}

__device__ inline unsigned short bf16_rn(float f)
{
    const unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
    return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

__device__ inline h8 load_frag(__amdgpu_buffer_rsrc_t src, int voff, int soff)
{
    return __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(src, voff, soff, 0));
}

// largest value / sum over the four lanes l, l^16, l^32, l^48 that share a query row
__device__ inline float max_row(float x)
{
    x = __builtin_fmaxf(x, __shfl_xor(x, 16));
    return __builtin_fmaxf(x, __shfl_xor(x, 32));
}
__device__ inline float sum_row(float x)
{
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
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
// What bounds it: few rows, the keys' way from memory (one row of 32768 keys, 28 heads on 4: 67 MB in 16 us; a large read
// reaches 6 TB/s here); more rows, the L2 (every 16 rows read all keys: 27 TB/s at 256 rows of 28 heads).  A wavefront has
// the 16 KB of a unit's keys and the 16 KB of its values in flight at once, eight wavefronts of a compute unit 256 KB.
template <int D, int RB, int NW>
__global__ __launch_bounds__(64 * NW)
void pasa_rows(const _Float16* __restrict__ q, const char* __restrict__ ws, const _Float16* __restrict__ kmean,
               _Float16* __restrict__ o, int lists, int list_rows, int Nq, int row0, int N, int causal, int nblk, int nsplit,
               int units, float coef, int tail_by_count, int io_bf16, const unsigned long long* gate,
               float* __restrict__ part_o, double* __restrict__ part_lr, size_t rows_all)
{
    constexpr int KS = D / 32;                   // k-steps of the first GEMM
    constexpr int CB = D / 16;                   // 16-channel blocks of O^T
    constexpr int ROWS = 16 * RB;
    constexpr int LD = D + 4;                    // LDS row of the merge, in floats
    constexpr int TILE_BYTES = 4 * T * D;        // K' tile then V tile
    __shared__ __attribute__((aligned(16))) float lds_o[NW * ROWS * LD];
    __shared__ double lds_r[NW][ROWS];
    __shared__ float lds_l[NW][ROWS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 15, g = lane >> 4;

    // grid: split fastest, then row block, then list of rows, then (batch, KV head)
    int idx = blockIdx.x;
    const int split = idx % nsplit;
    idx /= nsplit;
    const int blk = idx % nblk;
    idx /= nblk;
    const size_t grp = idx / lists;              // b * Hkv + hk
    if (gate != nullptr && gate[grp] == 0) return;   // adaptive start: nothing overflowed here
    const size_t list0 = (grp * lists + idx % lists) * (size_t)list_rows;   // first row of the list, in q and o
    const int p0 = blk * ROWS;
    int p1 = p0 + ROWS - 1;
    if (p1 > list_rows - 1) p1 = list_rows - 1;

    // keys seen by the block's rows: all up to the last position (causal), from the first position on only in part
    const int h0 = p0 / Nq, h1 = p1 / Nq;
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
    const int mv = (g * 32 + lq) * 16;

    h8 K[4 * KS], V[2 * CB];
    auto load_k = [&](int u) {
        const int base = (u >> 1) * TILE_BYTES + (u & 1) * (U * 16);
#pragma unroll
        for (int n = 0; n < 4 * KS; ++n) {                       // block n % 4, k-step n / 4
            const int i = (n % 4) >> 1, s = n & 1;
            K[n] = load_frag(tiles, kv, base + (n / 4) * (4 * T * 16) + i * (32 * 16) + s * (8 * 16));
        }
    };
    auto load_v = [&](int u) {
        const int base = (u >> 1) * TILE_BYTES + 2 * T * D + (u & 1) * (U * 2 * D);
#pragma unroll
        for (int n = 0; n < 2 * CB; ++n)                         // channel block n % CB, k-step n / CB
            V[n] = load_frag(tiles, vv, base + (n / CB) * (4 * D * 16) + (n % CB) * (16 * 16));
    };

    h8 Q[RB][KS];
    f4 O[RB][CB];
    float l[RB];
    double R[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        l[rb] = 0.f;
        R[rb] = -__builtin_inf();
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) O[rb][cb] = (f4)0.f;
    }

    if (u0 < ue) {
        load_k(u0);
        int last[RB];                            // last key that the lane's row sees
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int p = p0 + 16 * rb + lq;
            const bool real = p < list_rows;
            last[rb] = N - 1;
            if (causal && real && row0 + p % Nq < N - 1) last[rb] = row0 + p % Nq;
            const _Float16* src = q + (list0 + (real ? p : p0)) * D + 8 * g;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const h8 raw = *reinterpret_cast<const h8*>(src + 32 * ks);
                const h8 val = io_bf16 ? q_from_bf16(__builtin_bit_cast(u16x8, raw)) : raw;
                Q[rb][ks] = real ? val : (h8)(_Float16)0;
            }
        }
        f4 M[RB];                                // q . (mean rows) of eight tiles: see below
        int m8 = -1;
        for (int u = u0; u < ue; u += NW) {
            const int t = u >> 1;
            if ((t >> 3) != m8) {
                // the means of eight tiles: A rows 16 (t8 & 1) .. +15 of the mean block; lanes g = 0 (2) then hold the products
                // with the high parts of tiles 0-3 (4-7) of the eight, lanes g = 1 (3) those with the low parts
                m8 = t >> 3;
                h8 A[KS];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    A[ks] = load_frag(means, mv, (m8 >> 1) * (64 * D) + (m8 & 1) * (16 * 16) + ks * (4 * 32 * 16));
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    M[rb] = (f4)0.f;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks)
                        M[rb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[ks], Q[rb][ks], M[rb], 0, 0, 0);
                }
            }
            load_v(u);
            f4 S[RB][4];
#pragma unroll
            for (int n = 0; n < 4 * KS; ++n)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    S[rb][n % 4] = __builtin_amdgcn_mfma_f32_16x16x32_f16(K[n], Q[rb][n / 4], n < 4 ? (f4)0.f : S[rb][n % 4], 0, 0, 0);
            if (u + NW < ue) load_k(u + NW);

            const int e = t & 3, half = (t >> 2) & 1;
            const int tail = N - t * T;          // keys of this tile, when fewer than 128
            h8 P[RB][2];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const float me = e == 0 ? M[rb][0] : e == 1 ? M[rb][1] : e == 2 ? M[rb][2] : M[rb][3];
                float v = __shfl(me, lq + 32 * half) + __shfl(me, lq + 32 * half + 16) * 0.00048828125f;
                if (tail_by_count && tail < T) v *= (float)T * (1.0f / (float)tail);
                if (u * U + U - 1 > first_pos) {
#pragma unroll
                    for (int b = 0; b < 4; ++b)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (u * U + 32 * (b >> 1) + 16 * (g >> 1) + 8 * (b & 1) + 4 * (g & 1) + i > last[rb]) S[rb][b][i] = -__builtin_inff();
                }
                float mx = S[rb][0][0];
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i) mx = __builtin_fmaxf(mx, S[rb][b][i]);
                mx = max_row(mx);
                const bool unseen = mx == -__builtin_inff();     // the row sees no key of this unit
                const double lev = (double)mx + (double)coef * (double)v;
                const bool first = R[rb] == -__builtin_inf();
                float c = first ? (float)(lev - lev) : (float)(lev - R[rb]);      // first: 0, or NaN for a level that is none
                const bool move = !unseen && (first || c > CMAX);
                if (__builtin_amdgcn_ballot_w64(move && !first) != 0ull) {
                    const float r = (move && !first) ? __builtin_amdgcn_exp2f(-c * LOG2E) : 1.f;
                    l[rb] *= r;
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) O[rb][cb] *= r;
                }
                if (move) {
                    R[rb] = lev;
                    if (!first) c = 0.f;
                }
                const float nml = unseen ? 0.f : (c - mx) * LOG2E;
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const _Float16 ph = (_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(S[rb][b][i], LOG2E, nml));
                        P[rb][b >> 1][4 * (b & 1) + i] = ph;
                        l[rb] += (float)ph;
                    }
            }
#pragma unroll
            for (int n = 0; n < 2 * CB; ++n)
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
                    O[rb][n % CB] = __builtin_amdgcn_mfma_f32_16x16x32_f16(V[n], P[rb][n / CB], O[rb][n % CB], 0, 0, 0);
        }
    }

    // ---- the wavefronts' states brought to the highest of their levels and added ----
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        l[rb] = sum_row(l[rb]);
        if (g == 0) lds_r[wave][16 * rb + lq] = R[rb];
    }
    __syncthreads();
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        double rmax = -__builtin_inf();
#pragma unroll
        for (int w = 0; w < NW; ++w) rmax = __builtin_fmax(rmax, lds_r[w][16 * rb + lq]);
        const float wgt = R[rb] == -__builtin_inf() ? 0.f : __builtin_amdgcn_exp2f((float)(R[rb] - rmax) * LOG2E);
        if (g == 0) lds_l[wave][16 * rb + lq] = wgt * l[rb];
        float* dst = lds_o + (wave * ROWS + 16 * rb + lq) * LD + 4 * g;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) *reinterpret_cast<f4*>(dst + 16 * cb) = O[rb][cb] * wgt;
    }
    __syncthreads();
    for (int item = tid; item < ROWS * (D / 4); item += 64 * NW) {
        const int r = item / (D / 4), c4 = (item % (D / 4)) * 4;
        if (p0 + r >= list_rows) break;           // rows are in order: nothing real follows
        f4 acc = (f4)0.f;
        float ls = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            acc += *reinterpret_cast<const f4*>(lds_o + (w * ROWS + r) * LD + c4);
            ls += lds_l[w][r];
        }
        const size_t grow = list0 + p0 + r;
        if (nsplit > 1) {
            *reinterpret_cast<f4*>(part_o + ((size_t)split * rows_all + grow) * D + c4) = acc;
            if (c4 == 0) {
                double rmax = -__builtin_inf();
                for (int w = 0; w < NW; ++w) rmax = __builtin_fmax(rmax, lds_r[w][r]);
                part_lr[((size_t)split * rows_all + grow) * 2] = ls;
                part_lr[((size_t)split * rows_all + grow) * 2 + 1] = rmax;
            }
        } else {
            const float inv = 1.0f / ls;
            h4 out;
            u16x4 outb;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = acc[i] * inv;
                out[i] = (_Float16)x;
                outb[i] = bf16_rn(x);
            }
            if (io_bf16) *reinterpret_cast<u16x4*>(o + grow * D + c4) = outb;
            else *reinterpret_cast<h4*>(o + grow * D + c4) = out;
        }
    }
}

// Merge of the key splits of one call: per query row, the splits' stored outputs and sums are brought to the highest of
// their levels (the log-sum-exp rule on the absolute level a split's stored output refers to: m + Inva * F + Lc in
// pasa_fwd, R in pasa_rows) and added; then Algorithm 1's final quotient.  D / 8 threads of 8 channels per row, and SL
// such groups that share the row's splits.
template <int D, int SL>
__global__ __launch_bounds__(256) void pasa_merge_splits(const float* __restrict__ part_o, const double* __restrict__ part_lr,
                                                         _Float16* __restrict__ o, size_t rows_all, int nsplit, int io_bf16,
                                                         unsigned long long* nonfinite_o)
{
    constexpr int TPR = D / 8;                       // threads per row and group
    constexpr int RPB = 256 / (TPR * SL);            // rows per workgroup
    __shared__ float lds[SL > 1 ? 256 : 1][9];
    __shared__ double lds_max[SL > 1 ? RPB : 1][SL];
    const int tid = threadIdx.x, cl = tid % TPR, sl = (tid / TPR) % SL, rl = tid / (TPR * SL);
    const size_t row = (size_t)blockIdx.x * RPB + rl;
    const bool real = row < rows_all;
    const size_t grow = real ? row : rows_all - 1;
    const int c0 = cl * 8;
    double rmax = -__builtin_inf();
    for (int s = sl; s < nsplit; s += SL) rmax = __builtin_fmax(rmax, part_lr[((size_t)s * rows_all + grow) * 2 + 1]);
    if (SL > 1) {
        if (cl == 0) lds_max[rl][sl] = rmax;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SL; ++i) rmax = __builtin_fmax(rmax, lds_max[rl][i]);
    }
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    float lsum = 0.f;
#pragma unroll 4
    for (int s = sl; s < nsplit; s += SL) {
        const double r = part_lr[((size_t)s * rows_all + grow) * 2 + 1];
        if (r == -__builtin_inf()) continue;         // this split saw none of the row's keys (its output may not be written)
        const float wgt = __builtin_amdgcn_exp2f((float)(r - rmax) * LOG2E);
        lsum += wgt * (float)part_lr[((size_t)s * rows_all + grow) * 2];
        const f4* src = reinterpret_cast<const f4*>(part_o + ((size_t)s * rows_all + grow) * D + c0);
        const f4 a = src[0], b = src[1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[i] += wgt * a[i];
            acc[4 + i] += wgt * b[i];
        }
    }
    if (SL > 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) lds[tid][e] = acc[e];
        lds[tid][8] = lsum;
        __syncthreads();
        if (sl != 0) return;
#pragma unroll
        for (int i = 1; i < SL; ++i) {
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] += lds[tid + i * TPR][e];
            lsum += lds[tid + i * TPR][8];
        }
    }
    if (!real) return;
    const float inv = 1.0f / lsum;
    h8 out;
    u16x8 outb;
    unsigned n_bad = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float v32 = acc[e] * inv;
        out[e] = (_Float16)v32;
        outb[e] = bf16_rn(v32);
        const float fv = io_bf16 ? __uint_as_float((unsigned)outb[e] << 16) : (float)out[e];
        n_bad += (fv != fv || __builtin_fabsf(fv) == __builtin_inff()) ? 1u : 0u;
    }
    if (io_bf16) *reinterpret_cast<u16x8*>(o + grow * D + c0) = outb;
    else *reinterpret_cast<h8*>(o + grow * D + c0) = out;
    if (nonfinite_o != nullptr && n_bad) atomicAdd(nonfinite_o, (unsigned long long)n_bad);
}

template <int D, int SL>
void launch_merge(const void* part_o, const void* part_lr, void* o, size_t rows_all, int nsplit, int io_bf16,
                  unsigned long long* nonfinite_o, hipStream_t stream)
{
    constexpr int RPB = 256 / (D / 8 * SL);
    hipLaunchKernelGGL((pasa_merge_splits<D, SL>), dim3((unsigned)((rows_all + RPB - 1) / RPB)), dim3(256), 0, stream,
                       (const float*)part_o, (const double*)part_lr, (_Float16*)o, rows_all, nsplit, io_bf16, nonfinite_o);
}

template <int D, int RB, int NW>
hipError_t launch_rows(const PasaLaunch& p)
{
    const int G = p.Hq / p.Hkv, lists = p.Nq < 16 ? 1 : G, list_rows = p.Nq < 16 ? G * p.Nq : p.Nq;
    const int nblk = (list_rows + 16 * RB - 1) / (16 * RB);
    const int keys = p.causal && p.row0 < p.N - p.Nq ? p.row0 + p.Nq : p.N;
    const int all = (keys + U - 1) / U, units = (all + p.nsplit - 1) / p.nsplit;
    const int nsplit = (all + units - 1) / units;                 // none without keys
    const size_t rows_all = (size_t)p.B * p.Hq * p.Nq;
    hipLaunchKernelGGL((pasa_rows<D, RB, NW>), dim3((unsigned)((size_t)p.B * p.Hkv * lists * nblk * nsplit)), dim3(64 * NW), 0, p.stream,
                       (const _Float16*)p.q, (const char*)p.ws, (const _Float16*)p.kmean, (_Float16*)p.o, lists, list_rows, p.Nq, p.row0,
                       p.N, p.causal, nblk, nsplit, units, p.variant == PASA_K_DIRECT ? p.scale : p.inva,
                       p.variant == PASA_K_MIXED ? 1 : 0, p.io_bf16, p.gate, (float*)p.part_o, (double*)p.part_lr, rows_all);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nsplit == 1) return e;
    return pasa_launch_merge(p.part_o, p.part_lr, p.o, rows_all, p.d, nsplit, p.io_bf16, nullptr, p.stream);
}

}  // namespace

hipError_t pasa_launch_merge(const void* part_o, const void* part_lr, void* o, size_t rows_all, int d, int nsplit,
                             int io_bf16, unsigned long long* nonfinite_o, hipStream_t stream)
{
    const bool many = rows_all <= 4096 && nsplit > 2;
    if (d == 128)
        many ? launch_merge<128, 16>(part_o, part_lr, o, rows_all, nsplit, io_bf16, nonfinite_o, stream)
             : launch_merge<128, 1>(part_o, part_lr, o, rows_all, nsplit, io_bf16, nonfinite_o, stream);
    else
        many ? launch_merge<64, 16>(part_o, part_lr, o, rows_all, nsplit, io_bf16, nonfinite_o, stream)
             : launch_merge<64, 1>(part_o, part_lr, o, rows_all, nsplit, io_bf16, nonfinite_o, stream);
    return hipGetLastError();
}

hipError_t pasa_launch_rows(const PasaLaunch& p)
{
    return p.d == 128 ? launch_rows<128, 1, 8>(p) : launch_rows<64, 1, 8>(p);
}
