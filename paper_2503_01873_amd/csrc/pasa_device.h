// Device helpers that the kernels share.  Not installed.
#ifndef PASA_DEVICE_H
#define PASA_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

// Division of a number below 2^31 by a number that the host knows (at least 1): q = n * mul >> shift, exact, in three scalar
// instructions.  The compiler's division of two variables is a chain of forty through the vector unit; the kernels decode their
// workgroup's place with several, before their first load.
struct FastDiv {
    unsigned d, mul, shift;
    __host__ __device__ unsigned quotient(unsigned n) const { return (unsigned)(((unsigned long long)n * mul) >> shift); }
    __host__ __device__ unsigned rest(unsigned n, unsigned q) const { return n - q * d; }
};
inline FastDiv fast_div(unsigned d)
{
    unsigned s = 0;
    while ((1u << s) < d) ++s;                   // 2^s >= d > 2^(s-1): mul fits 32 bits, and n * (mul * d - 2^(31+s)) < 2^(31+s)
    return {d, (unsigned)(((1ull << (31 + s)) + d - 1) / d), 31 + s};
}

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

// bf16 inputs are converted to fp16 as they are loaded (the paper's remark on BF16 inputs): round to nearest even,
// values beyond the fp16 range become infinities.
__device__ inline h8 bf16x8_to_h8(u16x8 raw)
{
    h8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (_Float16)__uint_as_float((unsigned)raw[e] << 16);
    return out;
}

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));

// Two fp32 values -> a pair of bf16 / fp16, nearest even (v_cvt_pk_bf16_f32, v_cvt_pk_f16_f32; NaN stays NaN)
__device__ inline unsigned pack_bf16(float a, float b)
{
    const f2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf2));
}
__device__ inline unsigned pack_f16(float a, float b)
{
    const f2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, h2));
}


namespace {

constexpr int T = 128;          // keys per shift tile (s2 of the paper)
constexpr float LOG2E = 1.4426950408889634f;

// Value of x in the lane 32 away (lane l <-> lane l^32), without going through the LDS crossbar: the LDS pipe is
// saturated by the other wave group's fragment reads while this is needed.  v_permlane32_swap exchanges lanes 32-63
// of its first operand with lanes 0-31 of its second; with two copies of x that leaves [x_lo, x_lo] and [x_hi, x_hi].
// The s_nop cover the VALU-write -> permlane-read and permlane-write -> VALU-read wait states, which the compiler
// cannot see through inline assembly.
__device__ inline void halves32(float x, float& lo, float& hi)
{
    lo = x;
    hi = x;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1" : "+v"(lo), "+v"(hi));
}
// lanes 32-63 of a <-> lanes 0-31 of b.  Through the builtin, so that the compiler sees the reads: the operands here
// come straight from an MFMA, whose result registers must not be read before the instruction has written them all.
__device__ inline void swap32(float& a, float& b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}
__device__ inline float sum32(float x)
{
    float lo, hi;
    halves32(x, lo, hi);
    return lo + hi;
}
__device__ inline float max32(float x)
{
    float lo, hi;
    halves32(x, lo, hi);
    return __builtin_fmaxf(lo, hi);
}

// x of the even and of the odd one of each pair of 16-lane rows, in both; x of the lower and of the upper 32 lanes, in both
__device__ inline void rows16(float x, float& even, float& odd)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    even = __uint_as_float(r[0]);
    odd = __uint_as_float(r[1]);
}
__device__ inline void rows32(float x, float& low, float& high)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    low = __uint_as_float(r[0]);
    high = __uint_as_float(r[1]);
}
// largest value / sum over the four lanes l, l^16, l^32, l^48 that share a query row
__device__ inline float max_row(float x)
{
    float a, b;
    rows16(x, a, b);
    rows32(__builtin_fmaxf(a, b), a, b);
    return __builtin_fmaxf(a, b);
}
__device__ inline float sum_row(float x)
{
    float a, b;
    rows16(x, a, b);
    rows32(a + b, a, b);
    return a + b;
}
// the odd 16-lane rows of a <-> the even ones of b before them
__device__ inline void swap16(float& a, float& b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

__device__ inline float exp_nat(float x) { return __builtin_amdgcn_exp2f(x * LOG2E); }

__device__ inline h2 pack_rn(float a, float b)
{
    const f2 v = {a, b};
    return __builtin_convertvector(v, h2);     // v_cvt_pk_f16_f32: nearest-even
}

// a + b + acc with the two halves widened exactly (v_dot2_f32_f16 against ones)
__device__ inline float add_pair(h2 v, float acc)
{
    const h2 one = {(_Float16)1, (_Float16)1};
    return __builtin_amdgcn_fdot2(v, one, acc, false);
}

// P of a score, as the kernels make it: scale and offset in one fused multiply-add, the exponential rounded to fp16
__device__ inline float p_of(float score, float nml) { return (float)(_Float16)__builtin_amdgcn_exp2f(__builtin_fmaf(score, LOG2E, nml)); }

// The tiles on which a wavefront takes the maximum before it makes P: those before `end`.  A tile on which a row rises all the same is made again,
// which costs as much as the maximum of several.  Where such tiles follow one another within three, or that close behind the last one looked at, the
// next 2, 4, 8 and then 16 are looked at.  A single one changes nothing: rows of real values rise now and then, and the other wavefronts
// of the workgroup wait at its barriers for each tile that one of them looks at.
struct LookFirst {
    int end, tiles;
    __device__ inline void risen(int j)
    {
        if (end > j) return;                     // by the other block of rows of the same tile
        tiles = j - end >= 3 ? 0 : tiles == 0 ? 2 : tiles < 8 ? 2 * tiles : 16;
        end = j + 1 + tiles;
    }
};

// The largest of a lane's values of P; NaN where one of them is.
template <int N>
__device__ inline float largest_of(const h8 (&p)[N])
{
    h2 top[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        top[e] = h2{p[0][2 * e], p[0][2 * e + 1]};
#pragma unroll
        for (int i = 1; i < N; ++i) top[e] = __builtin_elementwise_maximum(top[e], h2{p[i][2 * e], p[i][2 * e + 1]});
    }
    const h2 t = __builtin_elementwise_maximum(__builtin_elementwise_maximum(top[0], top[1]), __builtin_elementwise_maximum(top[2], top[3]));
    const float a = (float)t[0], b = (float)t[1];
    return __builtin_elementwise_maximum(a, b);
}

// Scores of a block of 32 keys in the accumulator layout: -inf where key 8 (i / 4) + i % 4 (counted from the lane's first) is beyond
// `last`.  By bits: with a comparison per score the 64 results of a tile are wanted in scalar registers all at once, more than there are.
__device__ inline void mask_keys(f16v& s, int last)
{
    const int keep = last < 0 ? 0 : last > 31 ? 32 : last + 1;
    const unsigned beyond = (unsigned)(0xffffffffull << keep);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        unsigned m;                              // 0 or all ones; the builtin is turned into a comparison and a selection
        asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(beyond), "n"(8 * (i >> 2) + (i & 3)));
        s[i] = __uint_as_float((0xff800000u & m) | (__float_as_uint(s[i]) & ~m));
    }
}

// One wave-wide direct global -> LDS copy of 1 KiB: lane i moves 16 bytes from byte soff + 16*i of the buffer to
// ldst + 16*i.  soff and ldst must be wave-uniform (ldst travels in M0).
// OFF is an immediate added to both addresses, so a wave's consecutive pieces share one M0 value.
// The buffer form (buffer_load ... lds) is used rather than global_load_lds: the compiler treats the latter as a flat
// access that may touch LDS and from then on drains the LDS counter to zero before every use of an LDS fragment,
// which defeats the fragment prefetch of the GEMM loops.  soff has to lie within the buffer: the bounds check covers the
// lane's offset and the immediate, not the scalar offset.
template <int OFF>
__device__ inline void copy_1k_to_lds(__amdgpu_buffer_rsrc_t src, int soff, char* ldst, int lane)
{
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)ldst, 16, lane * 16, soff, OFF, 0);
}

// The output of a wavefront's 32 query rows goes through LDS (`mine`: 64 * D bytes that no other wavefront uses), so that a store
// writes 1 KiB of neighbouring bytes.  RB = 1, the 32x32 accumulators: lane (lq, g) holds channels 32 cb + 8 (e / 4) + 4 g + e % 4 of row lq.
// RB = 2, 16x16: channels 16 cb + 4 g + e of rows lq and 16 + lq.  value(rb, cb, e) is the one of element e.  dst: the first row; `rows` of them are
// real.  16-byte chunks are placed by row ^ chunk,
// against bank conflicts.  Straight from the accumulators, eight bytes a lane and a row apart, with the conversions of both types
// in line, the end of a workgroup of 256 rows took 3.5 us.
template <int D, int RB, bool BF16, class Value>
__device__ inline void store_rows_as(char* mine, Value value, _Float16* dst, int rows, int lane)
{
    asm volatile("" : "+v"(lane));               // no address is to be worked out before the main loop and kept through it
    constexpr int RR = 32 / RB, NE = 16 / (RB * RB);
    const int lq = lane & (RR - 1), g = lane / RR;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int cb = 0; cb < D / RR; ++cb)
#pragma unroll
            for (int e = 0; e < NE; e += 4) {
                uint2 x;
                x.x = BF16 ? pack_bf16(value(rb, cb, e), value(rb, cb, e + 1)) : pack_f16(value(rb, cb, e), value(rb, cb, e + 1));
                x.y = BF16 ? pack_bf16(value(rb, cb, e + 2), value(rb, cb, e + 3)) : pack_f16(value(rb, cb, e + 2), value(rb, cb, e + 3));
                const int chunk = RB == 1 ? 4 * cb + e / 4 : 2 * cb + (g >> 1);
                *reinterpret_cast<uint2*>(mine + (RR * rb + lq) * (2 * D) + ((chunk ^ (lq & 7)) * 16) + 8 * (g & 1)) = x;
            }
    __builtin_amdgcn_wave_barrier();             // a wavefront's LDS accesses are done in order
    asm volatile("" ::: "memory");
    constexpr int CH = D / 8, RPI = 64 / CH;     // chunks of a row, rows per store
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int r = i * RPI + lane / CH, c = lane % CH;
        const uint4 x = *reinterpret_cast<const uint4*>(mine + r * (2 * D) + ((c ^ (r & 7)) * 16));
        if (r < rows) *reinterpret_cast<uint4*>(dst + (size_t)r * D + 8 * c) = x;
    }
}
template <int D, int RB, class Value>
__device__ inline void store_rows(char* mine, Value value, _Float16* dst, int rows, int lane, int io_bf16)
{
    if (io_bf16) store_rows_as<D, RB, true>(mine, value, dst, rows, lane);
    else store_rows_as<D, RB, false>(mine, value, dst, rows, lane);
}

#define PASA_FENCE() __builtin_amdgcn_sched_barrier(0)

}  // namespace
#endif
