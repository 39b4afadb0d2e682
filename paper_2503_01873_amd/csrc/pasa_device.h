// Device helpers that the kernels share.  Not installed.
#ifndef PASA_DEVICE_H
#define PASA_DEVICE_H

#include <hip/hip_runtime.h>
#include <stdint.h>

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

// bf16 inputs are converted to fp16 as they are loaded (the paper's remark on BF16 inputs): round to nearest even,
// values beyond the fp16 range become infinities.
__device__ inline h8 bf16x8_to_h8(u16x8 raw)
{
    h8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (_Float16)__uint_as_float((unsigned)raw[e] << 16);
    return out;
}

__device__ inline h8 load_h8(const _Float16* p, int is_bf16)
{
    if (is_bf16) return bf16x8_to_h8(*reinterpret_cast<const u16x8*>(p));
    return *reinterpret_cast<const h8*>(p);
}

// fp32 -> bf16 bits, round to nearest even; NaN stays NaN
__device__ inline unsigned short f32_to_bf16_rn(float f)
{
    const unsigned u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
    return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f2 __attribute__((ext_vector_type(2)));


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

#define PASA_FENCE() __builtin_amdgcn_sched_barrier(0)

}  // namespace
#endif
