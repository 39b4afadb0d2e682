// PASA attention forward for gfx950: device kernels and their launchers.
//
// Two kernels per call.
//
//  pasa_prep_kv   Algorithm 1's pre-processing loop (Eq. (10), (11)) without forming the matrix M:
//                 per 128-key tile, the per-channel mean of K is taken exactly in fp64, K' = (K - beta*mean)*kscale
//                 is rounded once to fp16, and both K' and V are re-tiled so that the main kernel's LDS image of
//                 a tile is a straight copy whose MFMA fragments are single conflict-free 128-bit LDS reads.
//
//  pasa_fwd       Algorithm 1's main loops.  One workgroup = 8 wavefronts = 256 query rows; each wavefront owns
//                 32 query rows and sweeps the key tiles.  Both GEMMs are computed transposed, on
//                 v_mfma_f32_16x16x32_f16 (two blocks of 16 rows) or v_mfma_f32_32x32x16_f16 (one of 32; d = 64, STRICT16):
//                     S'^T = K' Q^T      (A = K' fragment from LDS, B = Q fragment held in registers)
//                     O^T += V^T P^T     (A = V^T fragment from LDS, B = P^T taken straight from the S'^T accumulators)
//                 In the transposed accumulator layout a lane holds a quarter (16 x 16: of two rows) or half of the keys of a query row, so
//                 the row statistics (pseudo-average Sbar', maximum m', sum l') are in-lane reductions plus an exchange
//                 between four or two lanes, and exp(S'-m') converted to fp16 is already the B operand of the second GEMM.
//
// Workspace: for every (batch, KV head, key tile) the K' tile followed by the V tile, so that one tile pair is
// one contiguous block that is copied to LDS verbatim with direct global->LDS loads, double buffered.
// For PASA_K_MIXED also, per (batch, KV head) and group of 16 key tiles, one "mean block": the per-channel mean over
// 128 key slots of the rounded K' of each of the 16 tiles, split into an fp16 high and an fp16 low part (times 2^11), laid out
// as a 32-row A operand (see pasa_prep_kv) -- by Eq. (12), (14) the pseudo-average of a score row is the query
// times that mean, which the main kernel takes for 16 tiles at a time on the matrix core.
// Tile layouts (one tile = 128 keys x D channels, fp16, 16-byte chunks):
//   K' tile: chunk index (c/8)*128 + n         holds channels 8*(c/8) .. +7 of key n
//   V  tile: chunk index ((n/16)*2 + h)*D + c  holds, for channel c, the 8 keys 16*(n/16) + {4h..4h+3, 8+4h..8+4h+3}
// The second layout is the key order in which a lane of the 32x32 accumulator holds its S'^T rows; with 16x16 the keys of a block are chosen to fit it.
//
// The matrix cores accumulate in fp32 in every variant; "fp16" quantities are rounded (nearest-even) where
// Algorithm 1 marks them.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>
#include <type_traits>
#include <utility>

#include "pasa_device.h"
#include "pasa_kernels.h"

namespace {

// ---------------------------------------------------------------------------------------------
// fp64 -> fp16 with a single rounding: truncate to fp32 (round to nearest, then step back if that
// rounded away from zero), make the fp32 "odd" when inexact, then
// let the hardware round fp32 -> fp16 to nearest-even.  fp32 has more than two extra bits, so the
// sticky bit makes the second rounding see exactly what a direct rounding would.
// ---------------------------------------------------------------------------------------------
__device__ inline _Float16 double_to_half_rn(double x)
{
    float f = (float)x;                         // nearest
    if ((double)f != x) {
        uint32_t u = __float_as_uint(f);
        if (__builtin_fabs((double)f) > __builtin_fabs(x)) u -= 1u;   // step the magnitude back: now truncated
        f = __uint_as_float(u | 1u);            // sticky bit
    }
    return (_Float16)f;
}

// The same for eight values.  Rounding twice, fp64 -> fp32 -> fp16, each to nearest, only goes wrong where the fp32 value
// is the midpoint of two fp16 values (13 last bits 0x1000; below 2^-14, where fp16 is subnormal, at other places): then,
// three chunks in ten of a wavefront with scaled keys of unit variance, the careful way above for all eight.
__device__ inline h8 doubles_to_halves_rn(const double (&x)[8])
{
    h8 out;
    unsigned off = 0xffffffffu;
    float least = 1.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float f = (float)x[e];
        out[e] = (_Float16)f;
        const unsigned d = (__float_as_uint(f) ^ 0x1000u) & 0x1fffu;
        off = d < off ? d : off;
        least = __builtin_fminf(least, __builtin_fabsf(f));
    }
    if (__builtin_amdgcn_ballot_w64(off == 0u || least < 0x1p-14f) != 0ull) {
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = double_to_half_rn(x[e]);
    }
    return out;
}

// Column sums of a wavefront whose lanes hold eight channels each of one or more keys, CH neighbouring lanes a key: by
// halves between lanes 32 and 16 apart (each keeps the channels of its side), then whole within a row of 16.  Lane l ends
// up with two channels, 4 (l / 32) + 2 (l / 16 % 2) and the next, of its eight.
__device__ inline void swap_doubles32(double& a, double& b)
{
    uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    const auto lo = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false), hi = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
    a = __builtin_bit_cast(double, uint2{lo[0], hi[0]});
    b = __builtin_bit_cast(double, uint2{lo[1], hi[1]});
}
__device__ inline void swap_doubles16(double& a, double& b)
{
    uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    const auto lo = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false), hi = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    a = __builtin_bit_cast(double, uint2{lo[0], hi[0]});
    b = __builtin_bit_cast(double, uint2{lo[1], hi[1]});
}
template <int ROR>
__device__ inline double rotated(double x)
{
    const uint2 v = __builtin_bit_cast(uint2, x);
    return __builtin_bit_cast(double, uint2{(unsigned)__builtin_amdgcn_update_dpp(0, (int)v.x, 0x120 + ROR, 0xf, 0xf, false),
                                            (unsigned)__builtin_amdgcn_update_dpp(0, (int)v.y, 0x120 + ROR, 0xf, 0xf, false)});
}
template <int CH>
__device__ inline void sum_columns(double (&s)[8], double& w0, double& w1)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        swap_doubles32(s[e], s[e + 4]);
        s[e] += s[e + 4];
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        swap_doubles16(s[e], s[e + 2]);
        s[e] += s[e + 2];
        s[e] += rotated<8>(s[e]);
        s[e] += rotated<4>(s[e]);
        if (CH == 2) s[e] += rotated<2>(s[e]);
    }
    w0 = s[0];
    w1 = s[1];
}

// ---------------------------------------------------------------------------------------------
// Pre-processing kernel.  256 threads; 2 * PASA_PREP_SPLIT blocks for each of the B*Hkv*ceil(N/128) tiles, numbered as below.
// plain_out != nullptr: write K' in the plain [.., N, D] layout instead (pasa_shift_keys).
// A ragged last tile is padded with zero keys and zero values in the workspace.
#ifndef PASA_PREP_SPLIT
#define PASA_PREP_SPLIT 4
#endif
constexpr unsigned PREP_ROW = 1u << 20;     // blocks in a row of the grid, where it has more than one

// One channel c of the two rows that key tile t owns in its "mean block" (a 32-row x D A operand per 16 tiles, in the
// K' tile's chunk order: chunk (c/8)*32 + row holds channels 8*(c/8)..+7 of row `row`).  Tile t of the group has its
// "high" row at 8*(t/4) + t%4 and its "low" row four rows further down: in the 32x32 accumulator layout the first kind
// of row lands in lanes 0-31 and the second in lanes 32-63 of the same accumulator register.  The last tile of a head
// also clears the rows of the tiles that do not exist.
__device__ inline void write_block_rows(_Float16* blocks, size_t head, int ntile, int t, int c, int D, _Float16 hi, _Float16 lo)
{
    const int nblk = (ntile + 15) / 16;
    const int t16 = t & 15, row = 8 * (t16 >> 2) + (t16 & 3);
    _Float16* blk = blocks + ((head * (size_t)nblk + (size_t)(t >> 4)) * 32) * D;
    blk[((size_t)(c / 8) * 32 + row) * 8 + (c % 8)] = hi;
    blk[((size_t)(c / 8) * 32 + row + 4) * 8 + (c % 8)] = lo;
    if (t == ntile - 1)
        for (int u = t16 + 1; u < 16; ++u) {
            const int ru = 8 * (u >> 2) + (u & 3);
            blk[((size_t)(c / 8) * 32 + ru) * 8 + (c % 8)] = (_Float16)0;
            blk[((size_t)(c / 8) * 32 + ru + 4) * 8 + (c % 8)] = (_Float16)0;
        }
}
// ---------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void pasa_prep_kv(const _Float16* __restrict__ k, const _Float16* __restrict__ v,
                                                    _Float16* __restrict__ wsout,
                                                    _Float16* __restrict__ plain_out, _Float16* __restrict__ k0out,
                                                    _Float16* __restrict__ kmean_out,
                                                    int N, FastDiv ntile_, double beta, double kscale, int shift_mode,
                                                    int in_bf16, const unsigned long long* gate, unsigned tiles, unsigned parts, unsigned group_log2, int y_off)
{
    // Workgroups are dealt round-robin to the 8 XCDs: blocks of a tile that read parts of the same 128-byte lines of K follow one
    // another on one XCD and share its L2, neighbouring tiles go to neighbouring XCDs.  `group` blocks of a tile come
    // together, all of them or the key blocks of all tiles before the value blocks (see the launch).
    // (Index of the block: where the grid has a second row, its rows hold PREP_ROW blocks, a multiple of 8.)
    const unsigned index = blockIdx.y * PREP_ROW + blockIdx.x;
    const unsigned per = (tiles + 7) >> 3;               // tiles of an XCD
    unsigned pos = index >> 3;
    if (pos >= per * parts) return;                      // the grid's last row is not full
    unsigned part = 0;
    if (pos >= per << group_log2) {
        pos -= per << group_log2;
        part = 1u << group_log2;
    }
    part += pos & ((1u << group_log2) - 1);
    const unsigned tile_ = (pos >> group_log2) * 8 + (index & 7);   // (batch, KV head, key tile)
    if (tile_ >= tiles) return;
    const int ntile = (int)ntile_.d;
    const unsigned head_ = ntile_.quotient(tile_);
    const size_t tile = tile_, head = head_;
    // adaptive start: nothing overflowed in this (batch, KV head), its shifted pass is not needed
    if (gate != nullptr && gate[head] == 0) return;

    // A tile's work is cut into 2*NS blocks: NS groups of D/NS channels of K (column means are per
    // channel, so the groups are independent) and NS groups of 128/NS keys of V.  The pass is bound by memory
    // latency and by fp64 arithmetic per thread, not by bandwidth, so it wants many small blocks.
    constexpr int NS = PASA_PREP_SPLIT;
    constexpr int DB = D / NS;           // channels of K per block
    constexpr int CH = DB / 8;           // 16-byte chunks per key within the group
    constexpr int KL = 256 / CH;         // key lanes
    constexpr int KPT = T / KL;          // keys per thread
    constexpr int TB = T / NS;           // keys of V per block
    constexpr size_t PSUM_BYTES = sizeof(double) * (2 * 4 + 1) * DB, VS_BYTES = sizeof(_Float16) * TB * (D + 8);
    __shared__ __attribute__((aligned(16))) char lds_raw[PSUM_BYTES > VS_BYTES ? PSUM_BYTES : VS_BYTES];

    const int t = (int)ntile_.rest(tile_, head_);
    const int nvalid = (N - t * T) < T ? (N - t * T) : T;    // keys of this tile (< 128 only in a ragged last tile)
    const size_t src_off = (head * (size_t)N + (size_t)t * T) * D;
    const int tid = threadIdx.x;

    // All loads of a thread are on the way at once: rows past the end are out of the buffer's bounds and come as zeros, bf16 is converted
    // afterwards.  With a branch for each of both, and the tile's place by division, 8 x 4 heads of 8192 keys took 53.5 us, now 49.5
    // (4.85 -> 5.4 TB/s); 14 x 5 heads of 5000 keys, d = 64, 8 % less.
    auto rows_of = [](const _Float16* x, size_t h, int rows) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(x) + h * (size_t)rows * D, 0, rows * (2 * D), 0x00020000);
    };
    auto load_row = [](__amdgpu_buffer_rsrc_t src, int row, int c8) {
        return __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(src, row * (2 * D) + 16 * c8, 0, 0));
    };
    const int by = (int)part + y_off;              // y_off = NS: only the value blocks are launched
    if (by >= NS) {
        // ---- values: keys [n0, n0 + TB) of the tile, all channels ----
        _Float16 (*vs)[D + 8] = reinterpret_cast<_Float16 (*)[D + 8]>(lds_raw);   // +8 halfs: rows 16 bytes apart in bank space
        const int n0 = (by - NS) * TB;
        constexpr int VCH = D / 8, VPT = TB * VCH / 256;
        const __amdgpu_buffer_rsrc_t vsrc = rows_of(v, head, N);
        h8 raw[VPT];
#pragma unroll
        for (int i = 0; i < VPT; ++i) raw[i] = load_row(vsrc, t * T + n0 + (tid + 256 * i) / VCH, (tid + 256 * i) % VCH);
        if (in_bf16) {
#pragma unroll
            for (int i = 0; i < VPT; ++i) raw[i] = bf16x8_to_h8(__builtin_bit_cast(u16x8, raw[i]));
        }
#pragma unroll
        for (int i = 0; i < VPT; ++i) *reinterpret_cast<h8*>(&vs[(tid + 256 * i) / VCH][8 * ((tid + 256 * i) % VCH)]) = raw[i];
        __syncthreads();
        _Float16* vdst = wsout + tile * (size_t)(2 * T * D) + T * D;
        const int chunk0 = (n0 / 16) * 2 * D;            // chunk ((n/16)*2 + h)*D + c; this block owns TB/16*2 values of (n/16)*2+h
        for (int chunk = tid; chunk < (TB / 16) * 2 * D; chunk += 256) {
            const int c = chunk % D;
            const int kh = chunk / D;
            const int nb = (kh >> 1) * 16 + (kh & 1) * 4;    // local key of the first of the 8
            h8 out;
#pragma unroll
            for (int e = 0; e < 8; ++e) out[e] = vs[nb + (e >> 2) * 8 + (e & 3)][c];
            *reinterpret_cast<h8*>(vdst + (size_t)(chunk0 + chunk) * 8) = out;
        }
        return;
    }

    // ---- keys: channels [cg*DB, cg*DB + DB) of the tile, all 128 keys ----
    double (*wsum)[4][DB] = reinterpret_cast<double (*)[4][DB]>(lds_raw);        // two sets of the wavefronts' column sums
    double* ragged = reinterpret_cast<double*>(wsum + 2);                        // [DB] means of a ragged tile
    const int cg = by;
    const int wave = tid >> 6, lane = tid & 63;
    const int c8 = tid % CH, kl = tid / CH;
    const int ch0 = cg * DB + 8 * c8;                    // first of this thread's 8 channels
    const int cw = 8 * c8 + 4 * (lane >> 5) + 2 * ((lane >> 4) & 1);   // first of the two channels it has the wavefront's sums of
    const __amdgpu_buffer_rsrc_t ksrc = rows_of(k, head, N);

    h8 kv[KPT];
    double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < KPT; ++i) kv[i] = load_row(ksrc, t * T + kl + KL * i, ch0 / 8);
    if (in_bf16) {
#pragma unroll
        for (int i = 0; i < KPT; ++i) kv[i] = bf16x8_to_h8(__builtin_bit_cast(u16x8, kv[i]));
    }
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += (double)kv[i][e];   // exact: fp16 values, at most 128 terms
    }
    double w0, w1;
    sum_columns<CH>(s, w0, w1);
    if ((lane & 15) < CH) {
        wsum[0][wave][cw] = w0;
        wsum[0][wave][cw + 1] = w1;
    }
    __syncthreads();
    // the tile's own key count, so that Eq. (14) holds for a ragged tile too; the matrix form needs the plain sum
    const bool divide = nvalid != T && shift_mode != PASA_PREP_MATRIX;
    if (divide) {                                        // one division a channel (a whole tile's is an exact scaling)
        if (tid < DB) ragged[tid] = ((wsum[0][0][tid] + wsum[0][1][tid]) + (wsum[0][2][tid] + wsum[0][3][tid])) / (double)nvalid;
        __syncthreads();
    }
    double mean[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {                        // every partial sum is exact in fp64: no order matters
        const double tot = (wsum[0][0][8 * c8 + e] + wsum[0][1][8 * c8 + e]) + (wsum[0][2][8 * c8 + e] + wsum[0][3][8 * c8 + e]);
        double val = shift_mode == PASA_PREP_MATRIX ? tot : divide ? ragged[8 * c8 + e] : tot * 0.0078125;
        if (shift_mode == PASA_PREP_MATRIX) val = __dmul_rn(kscale, val);
        if (shift_mode == PASA_PREP_MEAN) val = __dmul_rn(beta, val);
        // direct-bias recovery: the shift vector k0 = fp16(beta * mean) is itself an fp16 vector
        if (shift_mode == PASA_PREP_DIRECT) {
            const _Float16 k0h = double_to_half_rn(__dmul_rn(beta, val));
            val = (double)k0h;
            if (kl == 0) {
                k0out[tile * (size_t)D + ch0 + e] = k0h;
                // the main kernel reads the vector from the tile's "high" row of a mean block (below); the "low" row is zero
                if (kmean_out != nullptr) write_block_rows(kmean_out, head, ntile, t, ch0 + e, D, k0h, (_Float16)0);
            }
        }
        mean[e] = val;
    }
    double rs[8] = {0, 0, 0, 0, 0, 0, 0, 0};     // column sums of the ROUNDED K' over this thread's keys (exact in fp64)
#pragma unroll
    for (int i = 0; i < KPT; ++i) {
        const int n = kl + KL * i;
        double r[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if (shift_mode == PASA_PREP_MATRIX) {
                // K'^T = K^T M with M = a I + b (J - I) entrywise rounded to fp16 (Eq. (10), (11) as a GEMM):
                // sum_p M[p,q] K[p,c] = (a - b) K[q,c] + b sum_p K[p,c].  Here beta carries (a - b) and kscale
                // carries b; both products are exact in fp64 and the sum rounds once.
                r[e] = __dadd_rn(__dmul_rn(beta, (double)kv[i][e]), mean[e]);
            } else {
                // three separately rounded fp64 operations (no contraction): beta*mean, K - that, * kscale
                // (direct-bias recovery: K - k0 is exact)
                r[e] = __dmul_rn(__dsub_rn((double)kv[i][e], mean[e]), kscale);
            }
        }
        h8 out = doubles_to_halves_rn(r);
        if (n >= nvalid) out = (h8)(_Float16)0;  // padding keys: exact zeros
#pragma unroll
        for (int e = 0; e < 8; ++e) rs[e] += (double)out[e];
        if (plain_out != nullptr) {
            if (n < nvalid) *reinterpret_cast<h8*>(plain_out + src_off + (size_t)n * D + ch0) = out;
        } else {
            *reinterpret_cast<h8*>(wsout + tile * (size_t)(2 * T * D) + ((size_t)(ch0 / 8) * T + n) * 8) = out;
        }
    }
    if (kmean_out == nullptr || shift_mode == PASA_PREP_DIRECT) return;

    // ---- mean block: column sum of the rounded K' / 128 (an exact scaling), as an fp16 pair hi + lo ----
    sum_columns<CH>(rs, w0, w1);
    if ((lane & 15) < CH) {
        wsum[1][wave][cw] = w0;
        wsum[1][wave][cw + 1] = w1;
    }
    __syncthreads();
    if (tid < DB) {
        const double tot = (wsum[1][0][tid] + wsum[1][1][tid]) + (wsum[1][2][tid] + wsum[1][3][tid]);
        const double m128 = tot * 0.0078125;                 // 2^-7: exact
        // the low part is stored times 2^11 (undone when the two products are added): unscaled it is an fp16
        // subnormal for every mean below 0.125, and the matrix core reads those as zero
        const _Float16 hi = double_to_half_rn(m128);
        const _Float16 lo = double_to_half_rn((m128 - (double)hi) * 2048.0);
        write_block_rows(kmean_out, head, ntile, t, cg * DB + tid, D, hi, lo);
    }
}

// ---------------------------------------------------------------------------------------------
// Main kernel
// ---------------------------------------------------------------------------------------------
// (acc + a) + b, the same sum with two v_fma_mix_f32 (half * 1.0 + acc, the half read straight from its packed
// register).  v_dot2_f32_f16 takes its turn in the matrix pipeline: beside a wave that issues MFMAs back to back it
// holds its own wave for 24 cycles (a v_fma_mix_f32: 7) while costing the shared issue port little.  Where the vector
// part is short enough for that wait to show (STRICT16; MIXED since its pseudo-average moved to the matrix core) two of
// these are faster than one of those; in the other variants they are slower.  (The compiler folds fma(x, 1, acc) to
// an add with two separate conversions, hence the asm.)
__device__ inline float add_pair_mix(h2 v, float acc)
{
    asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel_hi:[1,0,0]" : "+v"(acc) : "v"(v));
    asm("v_fma_mix_f32 %0, %1, 1.0, %0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(acc) : "v"(v));
    return acc;
}

// exp of one half of a packed pair: (float)half * log2(e) in one v_fma_mix_f32 (the product rounded once, as a
// conversion followed by a multiplication would), then v_exp_f32
template <int HI>
__device__ inline float exp_nat_half(h2 v)
{
    float x;
    const float k = LOG2E;
    if (HI) asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(x) : "v"(v), "v"(k));
    else asm("v_fma_mix_f32 %0, %1, %2, 0 op_sel_hi:[1,0,0]" : "=v"(x) : "v"(v), "v"(k));
    return __builtin_amdgcn_exp2f(x);
}

// The same with an offset: 2 to the (float)half * log2(e) + off, a fused multiply-add
template <int HI>
__device__ inline float exp_off_half(h2 v, float off)
{
    float x;
    const float k = LOG2E;
    if (HI) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(x) : "v"(v), "s"(k), "v"(off));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(x) : "v"(v), "s"(k), "v"(off));
    return __builtin_amdgcn_exp2f(x);
}

__device__ inline f16v mma(h8 a, h8 b, f16v c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
__device__ inline f4 mma(h8 a, h8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

template <int... I, class F>
__device__ inline void for_constants(std::integer_sequence<int, I...>, F f) { (f(std::integral_constant<int, I>{}), ...); }

// A workgroup is 8 wavefronts and owns 256 query rows, 32 per wavefront.  Wavefronts 0-3 (group A) and 4-7
// (group B) sit pairwise on the four SIMDs and run the same program half a tile apart: time is cut into slots
// separated by workgroup barriers, and in every slot one group is in its matrix part while the other is in its
// vector part, so the MFMA pipe and the VALU of a SIMD are busy at the same time.
//
//   group A:  M(0) V(0) M(1) V(1) ...        group B:  -  M(0) V(0) M(1) ...
//   M(j) = [ O^T += V(j-1)^T P(j-1)^T ,  S'^T = K'(j) Q^T ]
//   V(j) = [ row statistics, global recovering scalars, exponentials -> P(j), row sum ]
//
// LDS holds two K' tiles and two V tiles; tile copies are direct global->LDS loads issued at the start of the vector
// parts, one to two slots before the first matrix part that reads them.
//
// Output accumulation.  STRICT16 keeps Algorithm 1's form: the tile product is rounded to fp16 and combined as
// O = fp16(e^{dm_j} * PV) + fp16(e^{dm_{j-1}} * O).  The fp32 variants accumulate the second GEMM directly onto the
// running output, which is stored at a scale of its own: O_j = e^{Lc_j} * Ostore_j.  The stored output is left alone
// and the tile's P takes the factor instead: with dp = dm_{j-1} and dc = dm_j of Algorithm 1's step 3,
// Lc_j = Lc_{j-1} + dp and P_j = fp16(exp(S' - m'_j + c_j)), c_j = dc - Lc_j, so Ostore_j = Ostore_{j-1} + P_j V_j and
// the running sum l is kept at the same scale (l += rowsum(P_j); the final quotient needs no factor).  c_j is the
// tile's level relative to the stored scale, which is the level of an earlier tile: c_j <= 0 unless the running
// maximum rises.  Only when c_j > 8 is a row's stored output and sum multiplied by e^{-c_j} (then Lc_j = dc, c_j = 0),
// a branch taken on a few tiles at the start of a row at most; so P <= e^8, far inside fp16, and a tile far below the
// running maximum underflows to zero by itself.  Against a rescale of the stored output on every tile this removes 64
// multiplications per tile and lane and three exponentials from the recovering scalars (3.7 % of the kernel time);
// the price is that P is Algorithm 1's exp(S' - m') times e^{c_j} rounded once, not exp(S' - m') rounded and then
// scaled, so outputs agree with a step-by-step evaluation to rounding, not bit for bit.  DIRECT (levels m' + c) and
// NAIVE16 (plain online softmax: P relative to the running maximum, dc = 0) use the same bookkeeping.
// MIXED and S16 keep the level of the stored output as one fp64 number R = m + inva * F + Lc, as the other kernels do, in which the
// reference level F cancels: P_j = fp16(exp(S' + inva * Sbar' - R)).  So the exponentials need no maximum; whether a row has
// risen is seen from its P (the largest of packed pairs, three at a time, nothing exchanged between lanes), and only a block of rows with such a
// row takes the maximum and makes P again.  Where rows rise on tile after tile, P made twice on all of them costs a fifth: the
// maximum is taken first on the first tile and on those that LookFirst names.  28 heads on 4, us, P first on every tile but the first / the maximum
// first on the 16 tiles behind every one made again / so (the maximum always: a tenth more on normal values): levels that rise by 3 per tile, 8192
// rows 509 / 471 / 472, by 9, 4096 rows not causal 269 / 237 / 241; normal values, 8192 rows 416 / 415 / 415; keys with outlier channels 421 / 436 / 422;
// 16384 rows, a key bias that changes every 1024 keys, 1585 / 1629 / 1592.
// Workgroups of two halves, whose chains are short, and MIXED at d = 64 take the maximum on every tile all the same: in the first tiles rows keep
// rising, and P made twice costs more there (us, without / so: 28 heads, 2048 rows 49.5 / 47.7; 8 heads, 4096 rows, not causal, 77.2 / 73.7, of 2500
// rows, d = 64, 50.1 / 47.0).  (DIRECT cannot: there a score may overflow where the tile's bias does not.)
//
// RB: the MFMAs.  RB = 1: one block of 32 rows, 32 x 32 x 16; RB = 2: two blocks of 16 rows, 16 x 16 x 32, each fragment of K' and V used twice
// in a row.  Both have the same rate and read as much LDS per product, but per product 16 x 16 x 32 moves half as many accumulators
// through the registers (twice as many operands, of half the width): with fragments from LDS and normal values a loop of nothing else reaches
// 1.68 PFLOP/s against 1.48, on zeros 2.37 against 2.40 (profiles/mfma_rate_of_two_shapes.txt).  Power is what bounds the long launches at d = 128, so they take it: 28 heads on 4, us, both
// sides in turn, 8192 rows 449 -> 403, 4096 rows not causal 233 -> 209; S16, 4096 rows 136 -> 124; DIRECT 129 -> 120; 1500 rows of 12000 keys
// 254 -> 242.  An MFMA holds the issue port though, and there are twice as many: where the vector part is the longer one (d = 64), or launches are short,
// 32 x 32 x 16 is faster (8 heads, d = 64, 2500 rows 50.1 / 53.6; STRICT16, 2 x 5 heads of 5000 rows, d = 64, 128 / 138, 12 heads on 2, 2257 rows, d = 128,
// 76.7 / 84.8).
//
// KSPL = 2: the workgroup owns 128 rows; both groups of wavefronts hold all of them, group A takes the even key tiles and
// group B the odd ones, each through a K' and a V buffer of its own, and B's state joins A's through LDS at the end (the rule of
// the key split).  A step (two slots) passes two tiles, so a workgroup's chain is half as long and there are twice as many
// workgroups: faster where the longest chain bounds the launch (28 heads on 4, causal, 1024 / 2048 rows 25.2 -> 17.9, 46.5 -> 39.7
// us), slower where the chip is full (8192 rows, kernels as they were, 446 -> 491 us: every tile is copied twice as often, and
// the start and the end of a workgroup come twice).
//
// What a workgroup needs to know its place in the launch (see the decode), worked out on the host: with its divisions in the kernel
// the first load went out 1.1 us after the workgroup's start.
struct FwdPlace {
    FastDiv nsplit, list, G;         // list: entries of a list that share a query tile
    int mode, span_log2;             // PASA_FWD_*; SHARED: 8 >> span_log2 groups, each on 1 << span_log2 XCDs
    int nwg, nqt, heads;             // workgroups without the key split, query tiles, B * Hq
    float inv_tail;                  // 1 / keys of the last tile
};
enum { PASA_FWD_OWN_GROUPS, PASA_FWD_SHARED, PASA_FWD_PLAIN };

template <int D, int VAR, bool CAUSAL, bool INSTR, int KSPL, int RB>
__global__ __launch_bounds__(512, 2)
void pasa_fwd(const _Float16* __restrict__ q, const char* __restrict__ ws, _Float16* __restrict__ o,
              const _Float16* __restrict__ kmean, FwdPlace at, int Nq, int row0, int N, float inva, float scale, int io_bf16,
              unsigned long long* ovf_s, unsigned long long* nonfinite_o, unsigned long long* ovf_group,
              const unsigned long long* gate, float* __restrict__ part_o, double* __restrict__ part_lr)
{

    constexpr int RR = 32 / RB;                  // rows of a block; keys or channels of a block of A
    constexpr int NE = 16 / (RB * RB);           // elements of an accumulator block that a lane holds
    constexpr int NG = 2 * RB;                   // lanes that share a query row; 16-byte chunks of a k-step
    constexpr int KS = D / (8 * NG);             // k-steps of S'^T = K' Q^T
    constexpr int CB = D / RR;                   // row blocks of O^T
    constexpr int KB = T / RR;                   // row blocks of S'^T
    constexpr int KK = T / (8 * NG);             // k-steps of O^T += V^T P^T
    using Acc = std::conditional_t<RB == 1, f16v, f4>;
    constexpr bool S16 = (VAR != PASA_K_MIXED && VAR != PASA_K_DIRECT);   // S' rounded to fp16 as it leaves the matrix core
    constexpr bool STRICT = (VAR == PASA_K_STRICT16);
    constexpr bool NAIVE = (VAR == PASA_K_NAIVE16);
    constexpr bool PACKED = (VAR == PASA_K_STRICT16 || VAR == PASA_K_S16);   // the rounded scores stay packed, two to a register
    constexpr bool DIRECT = (VAR == PASA_K_DIRECT);               // bias added back as scale * (q . k0), no pseudo-average
    // MIXED takes the pseudo-average as q . colmean(K') (Eq. (12), (14)) on the matrix core, 16 tiles at a time,
    // instead of summing 128 scores per row and tile on the vector unit
    // DIRECT takes q . k0 of the tiles the same way (their "mean block" holds the shift vectors, low rows zero)
    constexpr bool MSBAR = (VAR == PASA_K_MIXED || VAR == PASA_K_DIRECT);
    constexpr bool LEVEL = (VAR == PASA_K_MIXED || VAR == PASA_K_S16);     // the level of the stored output is kept as one number
    constexpr bool EAGER = KSPL == 2 || (D == 64 && MSBAR);     // LEVEL: the maximum on every tile all the same
    constexpr int KM_BYTES = 64 * D;                            // one mean block: 32 rows x D halfs
    constexpr int SB_OFF = 4 * (T * D * 2) + KM_BYTES;          // per-wave [16 tiles][32 rows] floats behind it
    constexpr int KT_BYTES = T * D * 2;                         // one K' (or V) tile
    constexpr int TILE_BYTES = 2 * KT_BYTES;                    // workspace stride: K' tile then V tile
    constexpr int CPW = KT_BYTES / 1024 / 8 * KSPL;             // 1 KiB copies per wave per K' (or V) tile
    constexpr int RW = 32, RWG = 256 / KSPL;
    static_assert(KSPL == 1 || !STRICT, "the fp16 state has no merge rule");
    static_assert(RB == 1 || !STRICT, "the fp16 state is that of one row");

    extern __shared__ __attribute__((aligned(1024))) char smem[];   // K'[2] then V[2]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = wave >> 2;
    const int lq = lane & (RR - 1), g = lane / RR;
    const int wcopy = KSPL == 1 ? wave : wave & 3;              // this wave's place among those that copy a tile
    const int jg = KSPL == 1 ? 0 : grp;                         // first tile of the wave's group, relative to j0

    // Work decode.  Workgroups are dispatched in index order and dealt round-robin to the 8 XCDs (index % 8), each
    // with its own L2.  Two goals: (1) every XCD walks its share longest-first -- the query tiles with the most key
    // tiles (the last ones when causal) first -- which keeps the tail of the launch short; (2) the query heads that
    // share one KV head run on the same XCD(s), so that K'/V tiles are fetched into as few L2s as possible.
    // A "group" is the set of Hq/Hkv query heads of one (batch, KV head).
    // Key split (nsplit > 1, for launches with too few workgroups to fill the chip): nsplit workgroups share one
    // (query tile, head); each sweeps a contiguous range of key tiles and leaves its per-row state (stored output, sum,
    // level) in part_o / part_lr for pasa_merge_splits.
    // How the workgroups of a launch reach the compute units was measured with a probe kernel (workgroups of this
    // kernel's LDS size that record their XCC, shader engine and compute unit and spin for a given time): within an XCD
    // they go to its four shader engines in strict rotation, in index order, and each waits for a compute unit of ITS
    // engine (8 per engine); a simulation of exactly that reproduces the probe's end times to 0.4 %.  With the items
    // simply longest first the engine that always gets the first of four carries 5 % more than the one that gets the
    // last (896 causal items of 2 .. 64 tile-steps end 4.5 % behind the mean).  So every other group of four
    // consecutive places of an XCD's list is taken backwards: the engines' loads even out and items that are
    // neighbours in the list stay neighbours in time, which keeps the query heads of a KV head on the same key tiles
    // at the same time (numberings that balance better but scatter the list ran slower: they lose that L2 reuse).
    const int nsplit = (int)at.nsplit.d;
    unsigned wg = at.nsplit.quotient(blockIdx.x);
    const int split = (int)at.nsplit.rest(blockIdx.x, wg);
    const unsigned x = wg & 7;
    {
        const unsigned r = wg >> 3, in_xcd = ((unsigned)at.nwg - x + 7) >> 3;             // workgroups of this XCD
        if ((r & 4) && (r | 3) < in_xcd) wg = ((r ^ 3) << 3) | x;
    }
    int qt, grp_id, hin;                    // query tile, group, head within group
    {
        const unsigned r = wg >> 3, span = 1u << at.span_log2;
        const unsigned i = at.mode == PASA_FWD_OWN_GROUPS ? r : at.mode == PASA_FWD_SHARED ? r * span + (x & (span - 1)) : wg;
        const unsigned up = at.list.quotient(i), rest = at.list.rest(i, up), g = at.G.quotient(rest);
        qt = at.nqt - 1 - (int)up;
        hin = (int)at.G.rest(rest, g);
        grp_id = at.mode == PASA_FWD_OWN_GROUPS ? x + 8 * g      // each XCD owns whole groups
                 : at.mode == PASA_FWD_SHARED ? x >> at.span_log2    // each group is spread over `span` XCDs: rest < G, g = 0
                                              : g;                   // plain longest-first order
    }
    // adaptive start: nothing overflowed in this (batch, KV head), its shifted pass is not needed (whole workgroup leaves)
    if (gate != nullptr && gate[grp_id] == 0) return;
    const size_t head = (size_t)grp_id * at.G.d + hin;           // b * Hq + hq
    const int ntile = (N + T - 1) / T;
    const int tail_keys = N % T;           // keys of a ragged last tile (0: none)
    const float inv_tail = at.inv_tail;

    // Query row r of the Nq rows given sits at sequence position row0 + r (causal: it sees keys <= its position).
    // Causal, both groups with rows: group A, which runs half a tile ahead, takes the later rows, whose keys reach a tile further.  Its
    // last matrix part is then the workgroup's last, half a tile before that of group B's with the later rows would be (28 heads on 4, us:
    // 3000 rows 81.6 -> 81.0, 4096 rows 128.5 -> 127.4, 8192 rows 467.1 -> 465.3; 2 x 16384 rows 3541 -> 3528).
    const int q0 = qt * RWG;
    const bool later_first = KSPL == 1 && CAUSAL && q0 + RWG / 2 < Nq;
    const int qw0 = q0 + (later_first ? wcopy ^ 4 : wcopy) * RW;
    bool wave_valid = qw0 < Nq;            // the wave owns at least one real row
    int last_row_wg = q0 + RWG - 1;
    if (last_row_wg > Nq - 1) last_row_wg = Nq - 1;
    int last_row_w = qw0 + RW - 1;
    if (last_row_w > Nq - 1) last_row_w = Nq - 1;
    auto tiles_seen = [&](int r) {         // key tiles a causal row at position row0 + r reaches
        const int t = (row0 + r) / T + 1;
        return t < ntile ? t : ntile;
    };
    // this workgroup's key tiles [j0, J_wg): all of the tiles its rows see, or -- split -- one range of them, cut at
    // multiples of 16 tiles so that a range starts with a mean block of its own
    const int J_all = CAUSAL ? tiles_seen(last_row_wg) : ntile;
    const int per16 = (int)at.nsplit.quotient(((J_all + 15) >> 4) + nsplit - 1);
    const bool splitting = !STRICT && nsplit > 1;      // STRICT16 is never launched split: its fp16 state has no merge rule
    const int j0 = splitting ? (split * per16 * 16 < J_all ? split * per16 * 16 : J_all) : 0;
    const int J_wg = splitting ? (j0 + per16 * 16 < J_all ? j0 + per16 * 16 : J_all) : J_all;
    int J_w = wave_valid ? (CAUSAL ? tiles_seen(last_row_w) : ntile) : 0;
    if (J_w > J_wg) J_w = J_wg;
    const int row = qw0 + lq;              // of the first block; those of a second are RR further on
    // (rows past the end compute on zero queries and are never stored)
    const int pos_w0 = row0 + qw0;         // position of the wave's first row

    const _Float16* qbase = q + head * Nq * D;
    const char* wsbase = ws + (size_t)grp_id * ntile * TILE_BYTES;
    // raw buffer over this (batch, KV head)'s tiles: at most 2048 tiles of 64 KiB, so every offset fits 32 bits
    const __amdgpu_buffer_rsrc_t wsbuf =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(wsbase), 0, ntile * TILE_BYTES, 0x00020000);

    // mean blocks of this (batch, KV head): block g serves tiles 16g .. 16g+15; one 1 KiB piece per wave (D = 64: waves 0-3)
    const int nblk16 = (ntile + 15) >> 4;
    const __amdgpu_buffer_rsrc_t kmbuf = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<_Float16*>(MSBAR ? kmean + (size_t)grp_id * nblk16 * (32 * D) : q), 0, MSBAR ? nblk16 * KM_BYTES : 0,
        0x00020000);
    auto issue_kmean = [&](int g) {
        if (MSBAR && wave * 1024 < KM_BYTES && g < nblk16)
            copy_1k_to_lds<0>(kmbuf, g * KM_BYTES + wave * 1024, smem + 4 * KT_BYTES + wave * 1024, lane);
    };
    // K' and V buffer of tile j: by turns, or -- key split within the workgroup -- one of each group's own
    auto buf = [&](int j) { return KSPL == 1 ? (j & 1) : grp; };
    auto issue_k = [&](int j) {
        const int src = j * TILE_BYTES;
        char* dst = smem + buf(j) * KT_BYTES;
#pragma unroll
        for (int i = 0; i < CPW; ++i) copy_1k_to_lds<0>(wsbuf, src + (wcopy * CPW + i) * 1024, dst + (wcopy * CPW + i) * 1024, lane);
    };
    // not past the last tile (a split with no keys, the second group of a single tile): the tile's offset is the scalar one,
    // which the buffer's bounds check leaves out
    if (j0 + jg < J_wg) issue_k(j0 + jg);
    issue_kmean(j0 >> 4);

    // Q fragments: B operand, lane (query lq, half lh) holds channels 16*ks + 8*lh .. +7.  The wavefront's rows come through LDS (the V
    // buffers, which are free until barrier 0) as 1 KiB copies, 16-byte chunks placed by row ^ chunk against bank conflicts: a
    // fragment's own load would touch 32 lines, and the first-level cache takes a line a clock for all eight wavefronts.
    {
        const __amdgpu_buffer_rsrc_t qbuf =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(qbase), 0, Nq * (2 * D), 0x00020000);
        constexpr int CH = D / 8;
        char* mine = smem + 2 * KT_BYTES + wave * (64 * D);
#pragma unroll
        for (int i = 0; i < D / 16; ++i) {
            const int r = i * (64 / CH) + lane / CH, at_row = qw0 + r < Nq ? qw0 + r : Nq - 1;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(qbuf, (__attribute__((address_space(3))) void*)(mine + i * 1024), 16,
                                                     at_row * (2 * D) + ((lane % CH) ^ (r & 7)) * 16, 0, 0, 0);
        }
    }
    // per-row state (one query row of each block per lane; the two or four lanes of a row hold copies)
    float m[RB], l[RB];              // fp32 variants
    float Lc[RB];                    // log of the scale of the stored output (DIRECT, NAIVE16)
    double R[RB];                    // LEVEL: level of the stored output, m + inva * F + Lc of Algorithm 1's state
    // STRICT: Algorithm 1's state; factors of the pending output combination, sum of the tile's P that goes with it
    _Float16 F16 = 0, m16 = 0, l16 = 0, ec16 = 0, ep16 = 0, lt16 = 0;
    h8 Pf[RB][KK];                   // P^T, B operand of the second GEMM
    Acc O[RB][CB];                   // fp32 variants: stored output; STRICT: product of the latest tile
    h2 O16[RB][CB][NE / 2];              // STRICT: running output
    unsigned long long n_ovf = 0;    // of the whole wavefront
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        l[rb] = Lc[rb] = 0.f;
        m[rb] = NAIVE ? -__builtin_inff() : 0.f;
        R[rb] = -__builtin_inf();
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) Pf[rb][kk] = (h8)(_Float16)0;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            O[rb][cb] = (Acc)0.f;
#pragma unroll
            for (int t = 0; t < NE / 2; ++t) O16[rb][cb][t] = (h2)(_Float16)0;
        }
    }

    // STRICT: fold the product of the latest tile (in O) into the running fp16 output
    auto fold16 = [&] {
        const h2 ec = {ec16, ec16}, ep = {ep16, ep16};
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int t = 0; t < NE / 2; ++t) {
                const h2 ot = pack_rn(O[0][cb][2 * t], O[0][cb][2 * t + 1]);
                const h2 a1 = ec * ot;                        // each packed op rounds to fp16 once; first tile: 1 * ot + 0 * 0
                const h2 a2 = ep * O16[0][cb][t];
                O16[0][cb][t] = a1 + a2;
            }
        // the running sum (step 4), each operation rounded: l = fp16(fp16(e^{dm_{j-1}} l) + fp16(e^{dm_j} l')); first tile: 0 + l'
        l16 = (_Float16)((_Float16)(ep16 * l16) + (_Float16)(ec16 * lt16));
    };

    // The copies of a slot are K'(jl + KSPL) and V(jl); each wave owns 2*CPW of their 1 KiB pieces.
    // A wave issues its pieces back to back at the start of its vector part (one wave-wide copy each, four of them sharing
    // M0 through immediate offsets).
    auto issue_piece = [&](int jl, auto piece_c) {
        constexpr int piece = decltype(piece_c)::value;       // 0 .. 2*CPW-1: K' pieces first, then V pieces
        constexpr int off = (piece % CPW) % 4 * 1024, base = (piece % CPW) / 4 * 4096;
        if (piece < CPW) {
            if (jl + KSPL < J_wg)
                copy_1k_to_lds<off>(wsbuf, (jl + KSPL) * TILE_BYTES + wcopy * (CPW * 1024) + base,
                                    smem + buf(jl + KSPL) * KT_BYTES + wcopy * (CPW * 1024) + base, lane);
        } else {
            if (jl < J_wg)
                copy_1k_to_lds<off>(wsbuf, jl * TILE_BYTES + KT_BYTES + wcopy * (CPW * 1024) + base,
                                    smem + 2 * KT_BYTES + buf(jl) * KT_BYTES + wcopy * (CPW * 1024) + base, lane);
        }
    };
    auto issue_slot = [&](int jl) {
        for_constants(std::make_integer_sequence<int, 2 * CPW>{}, [&](auto piece) { issue_piece(jl, piece); });
    };
    auto drain_copies = [&]() { __builtin_amdgcn_s_waitcnt(0x0F70); };   // vmcnt(0)

    // Barrier b ends slot b-1 and starts slot b.  Group A runs M(j) in slot 2j and V(j) in slot 2j+1; group B runs
    // M(j) in slot 2j+1 and V(j) in slot 2j+2.  Every wave issues its share of the copies K'(j+1), V(j) from its
    // vector part V(j) for group A (slot 2j+1) and V(j-1) for group B (slot 2j) -- the matrix part keeps its MFMA
    // chain free of them -- and drains them before the barrier that starts slot 2j+2, when group A reads them.
    drain_copies();
    h8 Qf[RB][KS];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const h8 raw = *reinterpret_cast<const h8*>(smem + 2 * KT_BYTES + wave * (64 * D) + (RR * rb + lq) * (2 * D) + (((NG * ks + g) ^ (lq & 7)) * 16));
            Qf[rb][ks] = row + RR * rb < Nq ? raw : (h8)(_Float16)0;
        }
    if (io_bf16) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) Qf[rb][ks] = bf16x8_to_h8(__builtin_bit_cast(u16x8, Qf[rb][ks]));
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);    // lgkmcnt(0): the rows have been read, the first values may take their place
    __syncthreads();                       // barrier 0: K'(0) is in LDS
    if (grp == 1) {
        if (KSPL == 1) issue_slot(j0);
        __syncthreads();                   // barrier 1: group B idles through slot 0
    }

    // Hand-offs between the parts of one wave.
    constexpr bool LAZY = !STRICT;   // fp32 variants: the recovering factor goes to P, not to the stored output
    // The row sums of a tile's P are not taken in the vector part that makes P, but by the matrix core in the matrix part that follows: one
    // more MFMA per k-step and row block of the second GEMM, P^T against a block of ones, accumulates the sums beside the stored output, at the same
    // scale (every row of the result is the sum).  28 heads of 4096 rows, not causal, 224.8 -> 213.3 us against additions between the MFMAs, DIRECT,
    // causal, 122.8 -> 121.2.
    // STRICT16 at d = 128 has no registers for it and adds them up between the MFMAs of the second GEMM.
    constexpr bool LSUM_DEFER = D == 128 && STRICT;
    constexpr bool LSUM_MFMA = !LSUM_DEFER;
    Acc Lacc[RB];
    float pl_d[2] = {0.f, 0.f};
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) Lacc[rb] = (Acc)0.f;
    constexpr float CMAX = 8.f;      // LAZY: P may exceed 1 by at most e^CMAX before the row re-references its scale
    constexpr float PMAX = 2980.f;   // LEVEL: the fp16 value below e^CMAX
    LookFirst look_first = {j0 + 1, 0};      // LEVEL, not EAGER: the tiles on which the maximum is taken first
    auto one_tile = [&](int rb) { return (CAUSAL && row0 + row + RR * rb < T) || N <= T; };      // the row sees a single tile

    // Both GEMMs run k-step by k-step: the fragments of a k-step go to the accumulator blocks in turn, so consecutive MFMAs never depend
    // on each other; with two row blocks each fragment is used twice, in alternating order, so that one operand stays from each MFMA to the next
    // (at 32 x 32 1.4 % faster than one dependent chain per accumulator block).  LDS fragments are fetched PF instructions ahead.
#ifndef PASA_PF
#define PASA_PF 3
#endif
    constexpr int PF = PASA_PF;
    constexpr int NM1 = KB * KS;     // fragments of the first GEMM
    constexpr int NM2 = CB * KK;     // fragments of the second GEMM
    auto sum_of_row = [](float x) { return RB == 1 ? sum32(x) : sum_row(x); };
    auto gemm1 = [&](int jt, Acc (&S)[RB][KB]) {   // S'^T of tile jt: 128 keys x 32 queries; fragment n: key block n % KB, k-step n / KB
        const _Float16* lds_k = reinterpret_cast<const _Float16*>(smem + buf(jt) * KT_BYTES);
        auto frag = [&](int n) {
            // 16 x 16: block 2i + s is keys 32i + {0..7, 16..23} + 8s, as in pasa_rows
            const int kb = n % KB, key = RB == 1 ? 32 * kb + lq : 32 * (kb >> 1) + 8 * (kb & 1) + 16 * (lq >> 3) + (lq & 7);
            return *reinterpret_cast<const h8*>(lds_k + ((NG * (n / KB) + g) * T + key) * 8);
        };
        h8 a[PF];
#pragma unroll
        for (int n = 0; n < PF; ++n) a[n] = frag(n);
        PASA_FENCE();
#pragma unroll
        for (int n = 0; n < NM1; ++n) {
            const int kb = n % KB, ks = n / KB;
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                const int rb = n & 1 ? RB - 1 - i : i;
                S[rb][kb] = mma(a[n % PF], Qf[rb][ks], ks == 0 ? (Acc)0.f : S[rb][kb]);
                PASA_FENCE();
            }
            if (n + PF < NM1) a[n % PF] = frag(n + PF);
            PASA_FENCE();
        }
    };
    auto gemm2 = [&](int jt) {   // (P V)^T of tile jt: D channels x 32 queries; runs during M(jt+1); fragment n: channel block n % CB, k-step n / CB
        const _Float16* lds_v = reinterpret_cast<const _Float16*>(smem + 2 * KT_BYTES + buf(jt) * KT_BYTES);
        unsigned one2 = 0x3c003c00u;             // a pair of ones
        if (LSUM_MFMA) asm volatile("" : "+v"(one2));      // made here each time, where there are registers, and not kept through the vector part
        auto frag = [&](int n) { return *reinterpret_cast<const h8*>(lds_v + ((NG * (n / CB) + g) * D + RR * (n % CB) + lq) * 8); };
        h8 a[PF];
#pragma unroll
        for (int n = 0; n < PF; ++n) a[n] = frag(n);
        PASA_FENCE();
#pragma unroll
        for (int n = 0; n < NM2; ++n) {
            const int cb = n % CB, kk = n / CB;
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                const int rb = n & 1 ? RB - 1 - i : i;
                O[rb][cb] = mma(a[n % PF], Pf[rb][kk], STRICT && kk == 0 ? (Acc)0.f : O[rb][cb]);
                PASA_FENCE();
            }
            if (n + PF < NM2) a[n % PF] = frag(n + PF);
            PASA_FENCE();
            if (LSUM_MFMA && cb == CB - 1) {
                const h8 ones = __builtin_bit_cast(h8, uint4{one2, one2, one2, one2});
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) Lacc[rb] = mma(ones, Pf[rb][kk], STRICT && kk == 0 ? (Acc)0.f : Lacc[rb]);
                PASA_FENCE();
            }
            if (LSUM_DEFER) {
                // 32 packed pairs over NM2 fragments
                constexpr int PER = 32 / NM2;
#pragma unroll
                for (int u = 0; u < PER; ++u) {
                    const int pr = n * PER + u;
                    const h2 p2 = {Pf[0][pr >> 2][2 * (pr & 3)], Pf[0][pr >> 2][2 * (pr & 3) + 1]};
                    pl_d[pr & 1] = add_pair_mix(p2, pl_d[pr & 1]);
                }
                PASA_FENCE();
            }
        }
        if (STRICT) {
            lt16 = (_Float16)(LSUM_MFMA ? Lacc[0][0] : sum32(pl_d[0] + pl_d[1]));
            pl_d[0] = pl_d[1] = 0.f;
        }
    };

    // The lane's number where it is rarely needed: what the compiler derives from it is not to be kept through the loop
    auto lane_again = [&] {
        int ln = lane;
        asm volatile("" : "+v"(ln));
        return ln;
    };

    // For where nothing reads these values before they are made again: without this the compiler keeps their registers, on the way past the
    // code that makes them, through all that comes before it
    auto forget_p = [&](int rb) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) asm volatile("" : "=v"(Pf[rb][kk]));
    };
    auto forget_product = [&] {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            asm volatile("" : "=v"(Lacc[rb]));
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) asm volatile("" : "=v"(O[rb][cb]));
        }
    };

    // Tiles that each group goes through, taken or not (KSPL = 1: to copy its share of them): as many, or group B one less
    const int n_a = KSPL == 1 ? J_wg - j0 : (J_wg - j0 + 1) / 2;
    const int n_b = KSPL == 2 ? (J_wg - j0) / 2 : n_a - (later_first && n_a > 0 && tiles_seen(q0 + RWG / 2 - 1) < J_wg ? 1 : 0);
    const int j_end = j0 + jg + KSPL * (grp == 0 ? n_a : n_b);
    for (int j = j0 + jg; j <= j_end; j += KSPL) {
        // =========================== matrix part M(j) ===========================
        const bool do_g2 = (j > j0 + jg && j - KSPL < J_w), do_g1 = (j < J_w);
        const bool tail = (tail_keys != 0) && (j == ntile - 1); // ragged last tile: padding keys are masked
        const bool diag = (CAUSAL && (j * T + T - 1 > pos_w0)) || tail;   // tile j needs the mask for this wave
        __builtin_amdgcn_s_setprio(1);
        // ---- pseudo-averages of the next 16 tiles: rows of A are the high and low parts of the tiles' mean keys ----
        if (MSBAR && ((j & 15) == jg || j == j0 + jg) && do_g1) {
            const int ln = lane_again(), lq = ln & (RR - 1), g = ln / RR;
            const _Float16* lds_km = reinterpret_cast<const _Float16*>(smem + 4 * KT_BYTES);
            // Half of the lanes hold q . hi of some tiles (32 x 32: those of g = 0, tile i in element i; 16 x 16: of g = 0 and 2, tile 8 ab + 2 g + e
            // in element e), the other half q . lo of the same; after the exchange their sum is a tile in each.
            float* sb = reinterpret_cast<float*>(smem + SB_OFF + wave * 2048);
#pragma unroll
            for (int ab = 0; ab < RB; ++ab) {
                Acc acc[RB];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const h8 mean = *reinterpret_cast<const h8*>(lds_km + ((NG * ks + g) * 32 + RR * ab + lq) * 8);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) acc[rb] = mma(mean, Qf[rb][ks], ks == 0 ? (Acc)0.f : acc[rb]);
                }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                    for (int e = 0; e < NE / 2; ++e) {
                        float x = acc[rb][e], y = acc[rb][e + NE / 2];
                        if (RB == 1) swap32(x, y);
                        else swap16(x, y);
                        const int tile = RB == 1 ? e + 8 * g : 8 * ab + 4 * (g >> 1) + 2 * (g & 1) + e;
                        sb[tile * 32 + RR * rb + lq] = x + y * 0.00048828125f;      // low parts are stored times 2^11
                    }
            }
        }
        // ---- pending product of tile j-1 ----
        if (do_g2) gemm2(j - KSPL);
        else if (STRICT && j == j0) forget_product();     // not past the wavefront's last tile: its product is folded in behind the loop
        // ---- S'(j) ----
        Acc S[RB][KB];                   // S'^T accumulators
        if (do_g1) gemm1(j, S);
        __builtin_amdgcn_s_setprio(0);
        if (KSPL == 1 && grp == 1) drain_copies();
        __syncthreads();
        // This wave's share of the tile copies first: they have the whole vector part to land (issued later, among the
        // exponentials, their latency showed at the drain before the next barrier: 3.8 % of the kernel's cycles).
        issue_slot(KSPL == 1 && grp ? j + 1 : j);
        if (MSBAR && (j & 15) == 8 + jg) issue_kmean((j >> 4) + 1);   // read from M(16 * ((j >> 4) + 1)) on, free since M(j - 8)
        PASA_FENCE();

        // =========================== vector part V(j) ===========================
        if (j < J_w) {
            const bool first = (j == j0 + jg);
            if (STRICT && do_g2) fold16();           // O <- fp16(e^{dm_j} PV) + fp16(e^{dm_{j-1}} O) for the product of tile j-1
            // ---- S' as stored: fp32, or rounded to fp16 ----
            // STRICT16 and S16 keep the rounded scores packed two per register; STRICT16 works on them with packed fp16
            // instructions (same roundings, half the instructions and registers)
            h2 Sh[RB][KB][NE / 2];
            if (INSTR) {
                // Only where there is something to count, and by the wavefront, a block at a time: a number per lane, and the 64 comparisons of
                // a tile all at once, took 152 (MIXED) to 187 (DIRECT) vector registers that were not there at d = 128.  28 heads on 4, 4096 rows,
                // us: MIXED 371 -> 126, DIRECT 455 -> 129, S16 157 -> 133, NAIVE16 204 -> 139; the adaptive start 210 -> 145, 512 rows 40 -> 30.
                // (Counted on every tile: 144, 150, 151, 159; d = 64, 14 x 5 heads, 2000 rows, adaptive 220 against 169.)
                float top[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < RB * KB * NE; ++i) top[i & 3] = __builtin_fmaxf(top[i & 3], __builtin_fabsf(S[i / (KB * NE)][i / NE % KB][i % NE]));
                if (__builtin_amdgcn_ballot_w64(__builtin_fmaxf(__builtin_fmaxf(top[0], top[1]), __builtin_fmaxf(top[2], top[3])) >= 65520.f) != 0ull) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int kb = 0; kb < KB; ++kb) {
                            asm volatile("" : "+v"(S[rb][kb]));
                            unsigned n = 0;
#pragma unroll
                            for (int e = 0; e < NE; ++e) n += (unsigned)__builtin_popcountll(__builtin_amdgcn_ballot_w64(__builtin_fabsf(S[rb][kb][e]) >= 65520.f));
                            asm volatile("" : "+s"(n));
                            n_ovf += n;
                        }
                }
            }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int e = 0; e < NE; ++e) {
                        if (PACKED) {
                            if (e & 1) Sh[rb][kb][e >> 1] = pack_rn(S[rb][kb][e - 1], S[rb][kb][e]);
                        } else if (S16) {
                            const float sv = (float)(_Float16)S[rb][kb][e];
                            S[rb][kb][e] = sv * scale;                   // NAIVE16, Eq. (2): static scaling after the GEMM
                        }
                    }
            // ---- pseudo-average over all 128 keys of the tile (before masking) ----
            float sbar[RB], cj[RB];          // cj: DIRECT, scale * (q . k0) of the tile
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                sbar[rb] = cj[rb] = 0.f;
                if (MSBAR) {
                    const float v = reinterpret_cast<const float*>(smem + SB_OFF + wave * 2048)[(j & 15) * 32 + RR * rb + lq];
                    if (DIRECT) cj[rb] = scale * v;                // the bias the shift removed from this tile's scores
                    else sbar[rb] = tail ? v * ((float)T * inv_tail) : v;   // stored per 128 key slots; a ragged last tile divides by its own key count
                }
            }
            if (PACKED) {
                // fp16 values summed in fp32 (as eight products of the matrix core with ones, which they lie right for: 4096 rows of S16 130.5 ->
                // 132.8 us, STRICT16 154.4 -> 156.2, since those wait behind the other wavefront's).
                // Padding keys of a ragged last tile have K' = 0 and add nothing; the divisor is the tile's own key count.
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    float ps[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int t = 0; t < KB * NE / 2; ++t) ps[t & 3] = add_pair_mix(Sh[rb][t / (NE / 2)][t % (NE / 2)], ps[t & 3]);
                    sbar[rb] = sum_of_row((ps[0] + ps[1]) + (ps[2] + ps[3])) * (tail ? inv_tail : 1.0f / T);
                }
            }
            // ---- mask: keys after the query (causal, diagonal tiles) or past the end (ragged last tile) ----
            if (diag) {
                const int ln = lane_again(), gn = ln / RR, posn = row0 + qw0 + (ln & (RR - 1));
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    int last_key = N - 1;
                    if (CAUSAL && posn + RR * rb < last_key) last_key = posn + RR * rb;
                    int key0 = j * T + (RB == 1 ? 4 * gn : 16 * (gn >> 1) + 4 * (gn & 1));
                    if (!CAUSAL) {
                        // Only the last tile is masked, nothing in the comparisons depends on j, and the compiler would take all 64 in front of
                        // the loop, into more scalar registers than there are: 0.7 us of every workgroup (28 heads on 4, 1024 rows 21.4 -> 19.5 us, 4096
                        // rows 221.1 -> 216.8; DIRECT, 4000 rows 217.4 -> 213.0)
                        last_key -= key0;
                        key0 = 0;
                        asm volatile("" : "+v"(last_key));
                    }
#pragma unroll
                    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                        for (int e = 0; e < NE; ++e) {
                            const int key = key0 + (RB == 1 ? 32 * kb + 8 * (e >> 2) + (e & 3) : 32 * (kb >> 1) + 8 * (kb & 1) + e);
                            if (!PACKED && key > last_key) S[rb][kb][e] = -__builtin_inff();
                            if (PACKED && (e & 1)) {         // a pair at once: taken apart, the scores would need twice the registers
                                const unsigned beyond = key > last_key ? (key - 1 > last_key ? 0xffffffffu : 0xffff0000u) : 0u;
                                unsigned& x = reinterpret_cast<unsigned&>(Sh[rb][kb][e >> 1]);
                                x = (0xfc00fc00u & beyond) | (x & ~beyond);
                            }
                        }
                }
            }
            // ---- local maximum m' ----
            auto row_max = [&](int rb) {
                float pm;                    // from four chains: one waits for each of its links
                if (PACKED) {
                    h2 mm[4];
#pragma unroll
                    for (int t = 0; t < KB * NE / 2; ++t) {
                        const h2 x = Sh[rb][t / (NE / 2)][t % (NE / 2)];
                        mm[t & 3] = t < 4 ? x : __builtin_elementwise_max(mm[t & 3], x);
                    }
                    const h2 top = __builtin_elementwise_max(__builtin_elementwise_max(mm[0], mm[1]), __builtin_elementwise_max(mm[2], mm[3]));
                    pm = __builtin_fmaxf((float)top[0], (float)top[1]);
                } else {
                    constexpr int PART = KB * NE / 4;
                    float part[4];
#pragma unroll
                    for (int i = 0; i < KB * NE; ++i) {
                        const float x = S[rb][i / NE][i % NE];
                        part[i / PART] = i % PART == 0 ? x : __builtin_fmaxf(part[i / PART], x);
                    }
                    pm = __builtin_fmaxf(__builtin_fmaxf(part[0], part[1]), __builtin_fmaxf(part[2], part[3]));
                }
                return RB == 1 ? max32(pm) : max_row(pm);
            };
            bool unseen[RB], resc[RB];       // resc, LAZY: this row re-references its stored output and sum to the level of tile j
            float top16 = 0.f;               // STRICT: m'
            float mref[RB], c_adj[RB];       // LAZY: log of the factor this tile's P carries (its level relative to the stored scale)
            float lc_resc[RB];               // LAZY: log of the factor that does it
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const float mx = LEVEL ? 0.f : row_max(rb);
                // A wave whose rows straddle a tile boundary (chunks not aligned to 32 rows) reaches tile j although its
                // first rows see none of it: those rows keep their state and add nothing.
                unseen[rb] = CAUSAL && diag && (row0 + row + RR * rb < j * T);
                // ---- reference level for exp: local m' (PASA), running max (plain FlashAttention) ----
                mref[rb] = unseen[rb] ? 0.f : mx;
                if (STRICT) top16 = mx;
                c_adj[rb] = lc_resc[rb] = 0.f;
                resc[rb] = false;
                // ---- fp32 variants: global recovering (step 3) and the factor of the output or of P now, before the
                // exponentials.  Only the running sum needs l'; the rest is a chain of dependent scalar operations whose
                // latency is hidden when the exponentials that follow can issue in between. ----
                // (values are read before they are chosen from: a choice between elements of arrays comes as branches)
                const bool out = unseen[rb];
                const float m0 = m[rb], Lc0 = Lc[rb];
                if (NAIVE) {
                    // plain online softmax (Eq. (4)-(8)) on the running maximum, the stored output handled as in MIXED:
                    // its log scale moves by m_{j-1} - m_j, P carries the factor, no per-tile rescale
                    const float mnew = __builtin_fmaxf(m0, mx);
                    const bool keep = first || out;
                    const float lcn = Lc0 + (m0 - mnew), c = -lcn;
                    const bool rs = !keep && c > CMAX;
                    resc[rb] = rs;
                    lc_resc[rb] = lcn;
                    c_adj[rb] = (keep || rs) ? 0.f : c;
                    Lc[rb] = first ? 0.f : out ? Lc0 : rs ? 0.f : lcn;
                    m[rb] = mnew;
                    mref[rb] = mnew;
                } else if (DIRECT) {
                    // ordinary online softmax on the level m' + c of this tile's maximum; same bookkeeping as below
                    const float lev = mx + cj[rb];
                    const float mn = __builtin_fmaxf(m0, lev);
                    const float dp = m0 - mn;
                    const float dc = lev - mn;
                    const bool keep = first || out;
                    const float lcn = Lc0 + dp, c = dc - lcn;
                    const bool rs = !keep && c > CMAX;
                    resc[rb] = rs;
                    lc_resc[rb] = -c;
                    c_adj[rb] = (keep || rs) ? 0.f : c;
                    Lc[rb] = first ? 0.f : out ? Lc0 : rs ? dc : lcn;
                    m[rb] = first ? lev : out ? m0 : mn;
                }
            }
            if (STRICT) {
                // Step 3 with every operation rounded to fp16, in the order Algorithm 1 states them; computed before the
                // exponentials and without branches (the first tile and rows that see nothing of the tile select their values
                // at the end) so that the latency of this chain is hidden.  The factors of the output combination go to ep16 /
                // ec16 (the pending product of tile j-1 has been folded in above).
                const _Float16 jm = (_Float16)(float)(j - j0), jn = (_Float16)(float)(j - j0 + 1), iv = (_Float16)inva;
                const _Float16 sb = (_Float16)sbar[0], mx = (_Float16)top16;
                const _Float16 Fn = (_Float16)((_Float16)((_Float16)(jm * F16) + sb) / jn);
                const _Float16 dpp = (_Float16)(iv * (_Float16)(F16 - Fn)), dpc = (_Float16)(iv * (_Float16)(sb - Fn));
                const _Float16 c1 = (_Float16)(m16 + dpp), c2 = (_Float16)(mx + dpc), mn = c1 > c2 ? c1 : c2;
                const _Float16 dp = (_Float16)((_Float16)(m16 - mn) + dpp), dc = (_Float16)((_Float16)(mx - mn) + dpc);
                const _Float16 ep = (_Float16)exp_nat((float)dp), ec = (_Float16)exp_nat((float)dc);
                const _Float16 one = 1, zero = 0;
                const bool out = unseen[0];
                F16 = first ? sb : out ? F16 : Fn;
                m16 = first ? mx : out ? m16 : mn;
                ep16 = first ? zero : out ? one : ep;    // unseen: O <- fp16(0 * 0) + fp16(1 * O)
                ec16 = first ? one : out ? zero : ec;
            }
            // what a row has stored so far, times r
            auto rescale = [&](int rb, float r) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int e = 0; e < NE; ++e) O[rb][cb][e] *= r;
#pragma unroll
                for (int e = 0; e < NE; ++e) Lacc[rb][e] *= r;
            };
            if (LAZY && !LEVEL && __builtin_amdgcn_ballot_w64(resc[0] || resc[RB - 1]) != 0ull) {
                // rare (the running maximum rose by more than CMAX above the stored scale); the pending product of
                // tile j-1 is already in O.  The empty asm keeps this a branch instead of 64 selects on every tile.
                asm volatile("" ::: "memory");
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) rescale(rb, resc[rb] ? exp_nat(lc_resc[rb]) : 1.f);
            }
            // ---- P = exp(S' - m' [+ c]) rounded to fp16 ----
            float nml[RB];
            auto exponentials = [&](int rb) {
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                    for (int t = 0; t < NE / 2; ++t) {
                        float e0, e1;
                        if (STRICT) {   // the difference is itself rounded to fp16 before the exponential
                            const _Float16 mh = (_Float16)mref[rb];      // exact: one of the fp16 scores (or 0)
                            const h2 d2 = Sh[rb][kb][t] - (h2){mh, mh};
                            e0 = exp_nat_half<0>(d2);
                            e1 = exp_nat_half<1>(d2);
                        } else if (PACKED) {
                            e0 = exp_off_half<0>(Sh[rb][kb][t], nml[rb]);
                            e1 = exp_off_half<1>(Sh[rb][kb][t], nml[rb]);
                        } else {        // exp(s - m) = 2^(s*log2e - m*log2e), one fused multiply-add per element
                            e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(S[rb][kb][2 * t], LOG2E, nml[rb]));
                            e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(S[rb][kb][2 * t + 1], LOG2E, nml[rb]));
                        }
                        const h2 p2 = pack_rn(e0, e1);
                        const int at = (kb * NE + 2 * t) / 8;
                        Pf[rb][at][(kb * NE + 2 * t) % 8] = p2[0];
                        Pf[rb][at][(kb * NE + 2 * t) % 8 + 1] = p2[1];
                    }
            };
            if (LEVEL) {
                // The scores of a tile stand for S' + inva * Sbar' (what the two correction terms of step 3 add up to: F cancels), so
                // P = exp(S' + inva * Sbar' - R) needs no maximum.  That a row has risen by more than CMAX above its stored output, or
                // has none yet (R = -inf), shows in P itself, and only then the maximum is taken, the row moved to the level of this
                // tile and P made again.  NaN, and with it the row, where the pseudo-average is not finite.
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    float off = __builtin_fmaf(sbar[rb], 0.f, (float)__builtin_fma((double)inva, (double)sbar[rb], -R[rb]));
                    if (CAUSAL && diag && unseen[rb]) off = 0.f;
                    nml[rb] = off * LOG2E;
                }
                float c[RB], up[RB];             // level of the tile above that of the stored output; offset of a row that moves to it
                double lev[RB];
                bool move[RB];
                auto look = [&](int rb) {
                    // a row that sees a single tile needs no pseudo-average, which may be infinite there
                    const float top = row_max(rb), bias = one_tile(rb) ? 0.f : sbar[rb], bad = (top + bias) * 0.f;
                    lev[rb] = (double)top + (double)inva * (double)bias;
                    c[rb] = (float)(lev[rb] - R[rb]) + bad;          // +inf for a row without keys so far
                    up[rb] = (bad - top) * LOG2E;
                    // not EAGER: as its own P shows it, which is rounded, so that a row does not go by what its neighbours do
                    move[rb] = !unseen[rb] && (EAGER ? c[rb] > CMAX : !(p_of(top, nml[rb]) <= PMAX));
                };
                auto settle = [&](int rb) {
                    if (!first) rescale(rb, move[rb] ? exp_nat(-c[rb]) : 1.f);      // (nothing is stored yet)
                    R[rb] = move[rb] ? lev[rb] : R[rb];
                    nml[rb] = move[rb] ? up[rb] : nml[rb];
                };
                if (EAGER || __builtin_expect(j < look_first.end, 0)) {
                    if (!EAGER) asm volatile("" ::: "memory");
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) look(rb);
                    if (__builtin_amdgcn_ballot_w64(move[0] || move[RB - 1]) != 0ull) {
                        asm volatile("" ::: "memory");
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) settle(rb);
                    }
                }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    exponentials(rb);
                    if (!EAGER && __builtin_expect(__builtin_amdgcn_ballot_w64(!(largest_of(Pf[rb]) <= PMAX)) != 0ull, 0)) {
                        asm volatile("" ::: "memory");
                        look_first.risen(j);
                        forget_p(rb);
                        look(rb);
                        settle(rb);
                        exponentials(rb);
                    }
                }
            } else {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    nml[rb] = (c_adj[rb] - mref[rb]) * LOG2E;
                    exponentials(rb);
                }
            }

            if (STRICT) forget_product();
        } else {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) forget_p(rb);
        }
        if (KSPL == 2 || grp == 0) drain_copies();
        __syncthreads();
    }
    if ((grp == 0) == (n_a == n_b)) __syncthreads();     // the barrier that the other group's last iteration ends with

    // level of the stored output; DIRECT, NAIVE16: running maximum and stored scale (exact in fp64)
    bool none[RB];
    double level[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        l[rb] = STRICT ? (float)l16 : Lacc[rb][0];      // every row of the block is the sum
        none[rb] = !(J_w > j0 + jg) || l[rb] == 0.f;
        // Not finite: a score or a pseudo-average left the range of its type, and the state must not be taken for one without keys.
        level[rb] = none[rb] ? -__builtin_inf() : LEVEL ? R[rb] : (double)m[rb] + (double)Lc[rb];
        if (!none[rb] && !__builtin_isfinite(level[rb])) level[rb] = __builtin_nan("");
    }
    // ---------------- key split within the workgroup: group B's state joins group A's ----------------
    if (KSPL == 2) {
        __syncthreads();                   // the tiles have been read
        static_assert(KSPL == 1 || 4 * RB * CB * NE * 64 * 4 <= 2 * KT_BYTES, "the exchange fits the K' tiles");
        f4* xo = reinterpret_cast<f4*>(smem) + (wave & 3) * (RB * CB * (NE / 4) * 64) + lane;
        double* xr = reinterpret_cast<double*>(smem + 2 * KT_BYTES) + (wave & 3) * (RB * 64) + lane;
        float* xl = reinterpret_cast<float*>(smem + 2 * KT_BYTES + 2048 * RB) + (wave & 3) * (RB * 64) + lane;
        if (grp == 1) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int e = 0; e < NE; e += 4)
                        xo[((rb * CB + cb) * NE + e) / 4 * 64] = f4{O[rb][cb][e], O[rb][cb][e + 1], O[rb][cb][e + 2], O[rb][cb][e + 3]};
                xr[rb * 64] = level[rb];
                xl[rb * 64] = none[rb] ? 0.f : l[rb];
            }
        }
        __syncthreads();
        if (grp == 0) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const double lev_b = xr[rb * 64];
                const double top = __builtin_fmax(level[rb], lev_b);
                // a state without keys weighs nothing, whatever its level; NaN stays NaN
                const float wa = none[rb] ? 0.f : __builtin_amdgcn_exp2f((float)(level[rb] - top) * LOG2E);
                const float wb = lev_b == -__builtin_inf() ? 0.f : __builtin_amdgcn_exp2f((float)(lev_b - top) * LOG2E);
                l[rb] = (none[rb] ? 0.f : l[rb] * wa) + xl[rb * 64] * wb;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int e = 0; e < NE; e += 4) {
                        const f4 x = xo[((rb * CB + cb) * NE + e) / 4 * 64];
#pragma unroll
                        for (int i = 0; i < 4; ++i) O[rb][cb][e + i] = O[rb][cb][e + i] * wa + x[i] * wb;
                    }
                level[rb] = top;
                none[rb] = l[rb] == 0.f;
            }
        } else {
            wave_valid = false;
        }
    }
    // ---------------- key split: leave the row state for the merge ----------------
    if (!STRICT && part_o != nullptr) {
        if (wave_valid) {
            const size_t rows_all = (size_t)at.heads * Nq;
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if (row + RR * rb >= Nq) continue;
                const size_t grow = (size_t)split * rows_all + head * Nq + row + RR * rb;        // row of the partial states
                if (g == 0) {
                    part_lr[grow * 2] = none[rb] ? 0.0 : (double)l[rb];
                    part_lr[grow * 2 + 1] = none[rb] ? -__builtin_inf() : l[rb] == l[rb] ? level[rb] : (double)l[rb];
                }
                if (!none[rb]) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                        for (int e = 0; e < NE; e += 4)
                            *reinterpret_cast<f4*>(part_o + grow * D + RR * cb + 2 * e + 4 * g) = f4{O[rb][cb][e], O[rb][cb][e + 1], O[rb][cb][e + 2], O[rb][cb][e + 3]};
                }
            }
        }
        if (INSTR) {
            if (ovf_s != nullptr && lane == 0 && n_ovf) atomicAdd(ovf_s, n_ovf);
            if (ovf_group != nullptr && lane == 0 && n_ovf) atomicAdd(ovf_group + grp_id, n_ovf);
        }
        return;
    }

    // ---------------- final normalisation and store ----------------
    unsigned long long n_bad = 0;
    if (wave_valid) {
        if (STRICT) fold16();
        float oscale[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) oscale[rb] = STRICT ? 0.f : 1.0f / l[rb];
        // fp32 variants: the fp32 quotient is rounded once, to the output type; STRICT16: the fp16
        // quotient of Algorithm 1's last line, converted when the output is bf16
        auto value = [&](int rb, int cb, int e) {
            return STRICT ? (float)(_Float16)(O16[rb][cb][e >> 1][e & 1] / l16) : O[rb][cb][e] * oscale[rb];
        };
        if (INSTR) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int e = 0; e < NE; ++e) {
                        const float x = value(rb, cb, e), fv = io_bf16 ? __uint_as_float(pack_bf16(x, 0.f) << 16) : (float)(_Float16)x;
                        n_bad += row + RR * rb < Nq && (fv != fv || __builtin_fabsf(fv) == __builtin_inff()) ? 1u : 0u;
                    }
        }
        // the tiles have been read by all wavefronts: both groups are past their last matrix parts (halves: where the wavefront
        // has just read the other group's output)
        store_rows<D, RB>(smem + wave * (64 * D * KSPL), value, o + (head * Nq + qw0) * D, Nq - qw0, lane, io_bf16);
    }
    if (INSTR) {
        if (ovf_s != nullptr && lane == 0 && n_ovf) atomicAdd(ovf_s, n_ovf);
        if (ovf_group != nullptr && lane == 0 && n_ovf) atomicAdd(ovf_group + grp_id, n_ovf);
        if (nonfinite_o != nullptr && n_bad) atomicAdd(nonfinite_o, n_bad);
    }
}

template <int D, int VAR, bool CAUSAL, bool INSTR, int KSPL = 1, int RB = (D == 128 && VAR != PASA_K_STRICT16 ? 2 : 1)>
hipError_t launch_fwd(const PasaLaunch& p)
{
    constexpr int RWG = 256 / KSPL;
    constexpr int LDS_BYTES = 4 * (T * D * 2) + ((VAR == PASA_K_MIXED || VAR == PASA_K_DIRECT) ? 64 * D + 8 * 2048 : 0);
    const int nqt = (p.Nq + RWG - 1) / RWG;
    const int nsplit = (VAR == PASA_K_STRICT16 || p.nsplit < 1) ? 1 : p.nsplit;   // fp16 state has no merge rule
    const dim3 grid((unsigned)(nqt * p.Hq * p.B * nsplit));
    auto kern = pasa_fwd<D, VAR, CAUSAL, INSTR, KSPL, RB>;
    // the dynamic LDS limit of this instantiation is raised once per device, not on every launch
    static std::atomic<unsigned long long> lds_limit_set{0ull};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(lds_limit_set.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        lds_limit_set.fetch_or(bit, std::memory_order_release);
    }
    const int G = p.Hq / p.Hkv, ngroups = p.B * p.Hkv, heads = p.B * p.Hq;
    FwdPlace at;
    at.nsplit = fast_div(nsplit);
    at.G = fast_div(G);
    at.mode = ngroups % 8 == 0 ? PASA_FWD_OWN_GROUPS
              : 8 % ngroups == 0 && (nqt * G) % (8 / ngroups) == 0 ? PASA_FWD_SHARED : PASA_FWD_PLAIN;
    at.list = fast_div(at.mode == PASA_FWD_OWN_GROUPS ? ngroups / 8 * G : at.mode == PASA_FWD_SHARED ? G : heads);
    at.span_log2 = at.mode != PASA_FWD_SHARED ? 0 : ngroups == 1 ? 3 : ngroups == 2 ? 2 : 1;
    at.nwg = nqt * heads;
    at.nqt = nqt;
    at.heads = heads;
    at.inv_tail = 1.0f / (float)(p.N % T ? p.N % T : T);
    hipLaunchKernelGGL(kern, grid, dim3(512), LDS_BYTES, p.stream, (const _Float16*)p.q, (const char*)p.ws,
                       (_Float16*)p.o, (const _Float16*)p.kmean, at, p.Nq, p.row0, p.N, p.inva, p.scale, p.io_bf16, p.overflow_s,
                       nsplit > 1 ? nullptr : p.nonfinite_o, p.overflow_group, p.gate,
                       nsplit > 1 ? (float*)p.part_o : nullptr, nsplit > 1 ? (double*)p.part_lr : nullptr);
    e = hipGetLastError();
    if (e != hipSuccess || nsplit == 1) return e;
    return pasa_launch_merge(p.part_o, p.part_lr, p.o, (size_t)p.B * p.Hq * p.Nq, D, nsplit, p.io_bf16, p.nonfinite_o, p.stream);
}

template <int D, int VAR>
hipError_t launch_fwd_cv(const PasaLaunch& p)
{
    const bool instr = p.overflow_s != nullptr || p.nonfinite_o != nullptr;
    if constexpr (D == 128 && VAR != PASA_K_STRICT16 && VAR != PASA_K_NAIVE16) {
        if (p.halves == 1 && !instr) return p.causal ? launch_fwd<D, VAR, true, false, 2, 1>(p) : launch_fwd<D, VAR, false, false, 2, 1>(p);
        if (p.halves == 2 && !instr) return p.causal ? launch_fwd<D, VAR, true, false, 2, 2>(p) : launch_fwd<D, VAR, false, false, 2, 2>(p);
    }
    if (p.causal) return instr ? launch_fwd<D, VAR, true, true>(p) : launch_fwd<D, VAR, true, false>(p);
    return instr ? launch_fwd<D, VAR, false, true>(p) : launch_fwd<D, VAR, false, false>(p);
}

template <int D>
hipError_t launch_fwd_d(const PasaLaunch& p)
{
    switch (p.variant) {
        case PASA_K_MIXED: return launch_fwd_cv<D, PASA_K_MIXED>(p);
        case PASA_K_STRICT16: return launch_fwd_cv<D, PASA_K_STRICT16>(p);
        case PASA_K_NAIVE16: return launch_fwd_cv<D, PASA_K_NAIVE16>(p);
        case PASA_K_S16: return launch_fwd_cv<D, PASA_K_S16>(p);
        case PASA_K_DIRECT: return launch_fwd_cv<D, PASA_K_DIRECT>(p);
    }
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t pasa_launch_prep(const void* k, const void* v, void* ws, void* plain_out,
                            int B, int Hkv, int N, int d, double beta, double kscale, int shift_mode, int in_bf16,
                            void* k0out, void* kmean_out, const unsigned long long* gate, hipStream_t stream)
{
    const int ntile = (N + T - 1) / T;
    const int y_off = k == nullptr ? PASA_PREP_SPLIT : 0;     // no keys given: the value blocks alone
    const unsigned parts = (v != nullptr && k != nullptr ? 2 : 1) * PASA_PREP_SPLIT;      // of a tile: key channel groups, then value key groups
    // A dimension of a grid holds fewer than 2^32 work items: beyond PREP_ROW blocks the launch goes on in a second dimension.
    const size_t tiles = (size_t)B * Hkv * ntile, blocks = (tiles + 7) / 8 * 8 * parts, row = PREP_ROW;
    const dim3 grid((unsigned)(blocks < row ? blocks : row), (unsigned)((blocks + row - 1) / row));
    // The key blocks take longer: first where the launch is a few rounds (8 heads of 4096 keys, d = 128, 256 tiles: 8.9 us, mixed
    // 11.6; 512 tiles 17.6 / 18.8), in longer ones mixed, so that reading, arithmetic and writing overlap (2048 tiles 58.9 /
    // 55.4; 14 x 5 heads of 9216 keys, d = 64: 82.9 / 80.3; both in plain order 63.5 and 92.5, before that 65.0 and 94.5).
    static_assert((PASA_PREP_SPLIT & (PASA_PREP_SPLIT - 1)) == 0, "blocks that come together are counted by shifts");
    const unsigned group = tiles < 1024 ? PASA_PREP_SPLIT : parts, group_log2 = (unsigned)__builtin_ctz(group);
    if (d == 128)
        hipLaunchKernelGGL(pasa_prep_kv<128>, grid, dim3(256), 0, stream, (const _Float16*)k, (const _Float16*)v,
                           (_Float16*)ws, (_Float16*)plain_out, (_Float16*)k0out, (_Float16*)kmean_out, N, fast_div(ntile), beta, kscale, shift_mode, in_bf16, gate, (unsigned)tiles, parts, group_log2, y_off);
    else
        hipLaunchKernelGGL(pasa_prep_kv<64>, grid, dim3(256), 0, stream, (const _Float16*)k, (const _Float16*)v,
                           (_Float16*)ws, (_Float16*)plain_out, (_Float16*)k0out, (_Float16*)kmean_out, N, fast_div(ntile), beta, kscale, shift_mode, in_bf16, gate, (unsigned)tiles, parts, group_log2, y_off);
    return hipGetLastError();
}

namespace {
__global__ void pasa_zero_u64(unsigned long long* p, int n)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0ull;
}
}  // namespace

hipError_t pasa_launch_zero(unsigned long long* p, int n, hipStream_t stream)
{
    hipLaunchKernelGGL(pasa_zero_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, p, n);
    return hipGetLastError();
}

hipError_t pasa_launch_fwd(const PasaLaunch& p)
{
    return p.d == 128 ? launch_fwd_d<128>(p) : launch_fwd_d<64>(p);
}
