// PASA attention for d = 64: pasa_fwd4, workgroups of four wavefronts that run free of one another.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <atomic>

#include "pasa_device.h"
#include "pasa_kernels.h"

namespace {

// A barrier that waits for no counter (the copies in flight are counted by hand) and that no memory access is moved across:
// the LDS reads before it have been used by then, those after it come after it.
__device__ inline void workgroup_barrier()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr float CMAX = 8.f;     // P may exceed 1 by at most e^CMAX before a row moves its stored output to a new level
constexpr float PMAX = 2980.f;  // the fp16 value below e^CMAX
constexpr int EARLY = 16;       // tiles at the start of a row in which it is likely to rise (see below)

// One workgroup = four wavefronts = 128 query rows of one head, 32 rows per wavefront; three workgroups share a compute
// unit and three wavefronts a SIMD.  The GEMMs are pasa_fwd's (32x32x16 MFMAs, transposed, fragments from LDS through a ring
// of three), but a wavefront goes through a tile in program order -- scores, softmax, output -- and what overlaps one
// wavefront's vector part with another's matrix part is that the three on a SIMD belong to workgroups that no barrier ties
// together.  pasa_fwd ties two wavefronts of a SIMD to opposite parts in slots of equal length; at d = 64 the softmax takes
// twice as long as the GEMMs, so that the matrix core waits for the longer part in every slot.
// LDS: K' of two tiles, V of one (V of tile j is asked for when its scores begin, K' of tile j + 1 right behind it), eight
// pseudo-averages per row: 52 KB, which is what lets three workgroups in.  Registers: 150 of the 168 that three
// wavefronts per SIMD leave.  The level of a row's stored output is one fp64 number, as in pasa_rows.  Row sums with
// v_dot2_f32_f16: the matrix core (P against ones) is faster on zeros (1163 against 1230 us) and slower on values (1519 / 1508 on
// the 14 x 5 heads of 9216 rows with resonant values, 1785 / 1713 with normal ones): power, not cycles, is what is short.
// That workload, pasa_fwd -> this kernel: 1624 -> 1508 us (1826 -> 1713 with normal values).
// MIXED makes P without the maximum of the tile, as pasa_fwd does (see there); a wavefront with a row that rises makes the scores again too,
// since there are no registers to keep them beside P (kept: spills, 283 -> 319 us on 14 x 5 heads of 5000 rows, causal).  us, both sides in turn, normal
// values: 14 x 5 heads of 9216 rows 1663 -> 1601, causal 5000 rows 284 -> 274; 16 heads of 8192 rows 315 -> 295, causal 16000 rows 575 -> 554.
// In the first tiles of a row, where rows keep rising, P would be made twice on most of them: there the maximum is taken first (resonant
// values, us, without the maximum from the second tile on / from the 9th / 17th / 33rd: 4 x 16 heads of 930 rows 39.8 / 36.2 / 36.2 / 36.2, 4 x 5 heads of
// 3786 rows, causal, 69.9 / 69.4 / 68.8 / 67.8; 2 x 5 heads of 9216 rows, normal values, 273.1 / 273.9 / 274.4 / 277.3, the maximum always 286.5).
// So it is later where rows of the wavefront rise on tile after tile, as LookFirst says (14 x 5 heads of 5000 rows, causal, us, not so / on the 16 tiles
// behind every one on which a row rose / so: levels that rise by 1 per tile 329 / 303 / 312, by 3 349 / 309 / 313; normal values 289 / 289 / 290).
// 64 rows per wavefront and two workgroups to a compute unit on top of it (half the LDS reads): 1 % faster on the 9216 rows,
// 4 to 20 % slower on all smaller calls.
template <bool CAUSAL, bool DIRECT>
__global__ __launch_bounds__(256, 3)
void pasa_fwd4(const _Float16* __restrict__ q, const char* __restrict__ ws, _Float16* __restrict__ o,
               const _Float16* __restrict__ kmean, int Hq, int Hkv, int Nq, int row0, int N, int nqt, float coef,
               int io_bf16, const unsigned long long* gate, int nsplit, float* __restrict__ part_o,
               double* __restrict__ part_lr)
{
    constexpr int D = 64;
    constexpr int KS = D / 16;                   // k-steps of S'^T = K' Q^T
    constexpr int CB = D / 32;                   // 32-channel row blocks of O^T
    constexpr int KT_BYTES = T * D * 2;          // one K' (or V) tile
    constexpr int TILE_BYTES = 2 * KT_BYTES;
    constexpr int CPW = KT_BYTES / 1024 / 4;     // 1 KiB copies per wavefront and tile
    constexpr int RW = 32, RWG = 128;
    constexpr int V_OFF = 2 * KT_BYTES, SB_OFF = 3 * KT_BYTES;

    extern __shared__ __attribute__((aligned(1024))) char smem[];   // K' of two tiles, V of one, pseudo-averages

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, lh = lane >> 5;

    // Workgroups are dealt round-robin to the 8 XCDs, each with an L2 of its own.  Equal items: every XCD gets a contiguous
    // range of them, the row tiles of a head after one another.  Causal: the longest first; every XCD its own heads where
    // they divide evenly.
    int qt, split;
    size_t head;                                 // b * Hq + hq
    const int G = Hq / Hkv;
    {
        const int x = blockIdx.x & 7, r = blockIdx.x >> 3, whole = gridDim.x >> 3, rest = gridDim.x & 7;
        const int lists = gridDim.x / nqt;       // (head, split) pairs
        int hs;
        if (!CAUSAL) {
            const int w = x * whole + (x < rest ? x : rest) + r;
            qt = w % nqt;
            hs = w / nqt;
        } else if (lists % 8 == 0) {
            const int per = lists >> 3;
            qt = nqt - 1 - r / per;
            hs = x * per + r % per;
        } else {
            qt = nqt - 1 - blockIdx.x / lists;
            hs = blockIdx.x % lists;
        }
        split = hs % nsplit;
        head = hs / nsplit;
    }
    const size_t grp = head / G;                 // b * Hkv + hk
    if (gate != nullptr && gate[grp] == 0) return;
    const int ntile = (N + T - 1) / T;

    const int qw0 = qt * RWG + wave * RW;
    int last_row_wg = qt * RWG + RWG - 1;
    if (last_row_wg > Nq - 1) last_row_wg = Nq - 1;
    int last_row_w = qw0 + RW - 1;
    if (last_row_w > Nq - 1) last_row_w = Nq - 1;
    auto tiles_seen = [&](int r) {
        const int t = (row0 + r) / T + 1;
        return t < ntile ? t : ntile;
    };
    const int J_all = CAUSAL ? tiles_seen(last_row_wg) : ntile;
    const int per = ((J_all + 7) / 8 + nsplit - 1) / nsplit * 8;      // tiles of a split, cut at multiples of 8
    const int j0 = split * per < J_all ? split * per : J_all;
    const int J_wg = j0 + per < J_all ? j0 + per : J_all;
    int J_w = qw0 < Nq ? (CAUSAL ? tiles_seen(last_row_w) : ntile) : 0;
    if (J_w > J_wg) J_w = J_wg;
    const int row = qw0 + lq;
    const bool row_valid = row < Nq;
    const int pos_w0 = row0 + qw0;
    int last_key = N - 1;
    if (CAUSAL && row0 + row < last_key) last_key = row0 + row;

    const __amdgpu_buffer_rsrc_t wsbuf = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(ws) + grp * (size_t)ntile * TILE_BYTES, 0, ntile * TILE_BYTES, 0x00020000);
    auto issue_k = [&](int j, int buf) {
        char* dst = smem + buf * KT_BYTES + wave * (CPW * 1024);
        const int src = j * TILE_BYTES + wave * (CPW * 1024);
#pragma unroll
        for (int i = 0; i < CPW; ++i) copy_1k_to_lds<0>(wsbuf, src + i * 1024, dst + i * 1024, lane);
    };
    auto issue_v = [&](int j) {
        char* dst = smem + V_OFF + wave * (CPW * 1024);
        const int src = j * TILE_BYTES + KT_BYTES + wave * (CPW * 1024);
#pragma unroll
        for (int i = 0; i < CPW; ++i) copy_1k_to_lds<0>(wsbuf, src + i * 1024, dst + i * 1024, lane);
    };

    h8 Qf[KS];
    f16v O[CB];
    float l4[4] = {0.f, 0.f, 0.f, 0.f};          // row sum of P over this lane's keys, in four parts
    double R = -__builtin_inf();                 // absolute level of the stored output
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) O[cb] = (f16v)0.f;
    if (j0 < J_wg) {
        issue_k(j0, j0 & 1);
        const __amdgpu_buffer_rsrc_t qbuf =             // rows past the end come as zeros
            __builtin_amdgcn_make_buffer_rsrc(const_cast<_Float16*>(q + head * Nq * D), 0, Nq * (2 * D), 0x00020000);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            Qf[ks] = __builtin_bit_cast(h8, __builtin_amdgcn_raw_buffer_load_b128(qbuf, row * (2 * D) + 16 * lh, 32 * ks, 0));
        if (io_bf16) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) Qf[ks] = bf16x8_to_h8(__builtin_bit_cast(u16x8, Qf[ks]));
        }
    }
    const int nblk16 = (ntile + 15) >> 4;
    const _Float16* km = kmean + grp * (size_t)nblk16 * (32 * D);
    float* sb = reinterpret_cast<float*>(smem + SB_OFF + wave * 1024);       // [8 tiles][32 rows]

    constexpr int PF = 3;
    LookFirst look_first = {j0 + EARLY, 0};
    for (int j = j0; j < J_wg; ++j) {
        // pseudo-averages of the next eight tiles (a block of A holds sixteen: the other half is not kept)
        if ((j & 7) == 0 && j < J_w) {
            const _Float16* blk = km + (size_t)(j >> 4) * (32 * D);
            f16v acc = (f16v)0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const h8*>(blk + ((2 * ks + lh) * 32 + lq) * 8), Qf[ks], acc, 0, 0, 0);
            const int hi8 = (j >> 3) & 1;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float x = hi8 ? acc[i + 8] : acc[i], y = hi8 ? acc[i + 12] : acc[i + 4];
                swap32(x, y);
                sb[(i + 4 * lh) * 32 + lq] = x + y * 0.00048828125f;
            }
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);      // vmcnt(0): this wavefront's share of K'(j)
        workgroup_barrier();                     // K'(j) is there; V(j-1) and K'(j-1) have been read
        PASA_FENCE();
        issue_v(j);
        // Beside the last tile it is fetched once more, into the buffer that nothing reads again: the tile's offset is the
        // scalar one, which the buffer's bounds check leaves out, and the number of copies in flight stays the same.
        issue_k(j + 1 < J_wg ? j + 1 : j, (j + 1) & 1);
        PASA_FENCE();
        h8 Pf[8];
        if (j < J_w) {
            f16v S[4];
            auto scores = [&] {
                const _Float16* lds_k = reinterpret_cast<const _Float16*>(smem + (j & 1) * KT_BYTES);
                auto frag = [&](int n) { return *reinterpret_cast<const h8*>(lds_k + ((2 * (n / 4) + lh) * T + 32 * (n % 4) + lq) * 8); };
                h8 a[PF];
#pragma unroll
                for (int n = 0; n < PF; ++n) a[n] = frag(n);
                PASA_FENCE();
#pragma unroll
                for (int n = 0; n < 4 * KS; ++n) {
                    S[n % 4] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[n % PF], Qf[n / 4], n < 4 ? (f16v)0.f : S[n % 4], 0, 0, 0);
                    PASA_FENCE();
                    if (n + PF < 4 * KS) a[n % PF] = frag(n + PF);
                    PASA_FENCE();
                }
                if ((CAUSAL && j * T + T - 1 > pos_w0) || N - j * T < T) {
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb) mask_keys(S[kb], last_key - (j * T + 32 * kb + 4 * lh));
                }
            };
            float v = sb[(j & 7) * 32 + lq];
            if (!DIRECT && N - j * T < T) v *= (float)T * (1.0f / (float)(N - j * T));
            // By position: the scores of keys that the row sees may all have overflowed to -inf
            const bool unseen = last_key < j * T;
            float nml;
            auto exponentials = [&] {
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int t2 = 0; t2 < 8; ++t2) {
                        const h2 p2 = pack_rn(__builtin_amdgcn_exp2f(__builtin_fmaf(S[kb][2 * t2], LOG2E, nml)),
                                              __builtin_amdgcn_exp2f(__builtin_fmaf(S[kb][2 * t2 + 1], LOG2E, nml)));
                        Pf[2 * kb + (t2 >> 2)][2 * (t2 & 3)] = p2[0];
                        Pf[2 * kb + (t2 >> 2)][2 * (t2 & 3) + 1] = p2[1];
                    }
            };
            // Rows that `rises` holds for, and that see keys of the tile, move to its level: the maximum of its scores and their bias.  A
            // row that sees a single tile needs no bias, which may be infinite.  nml is NaN, and with it the row, where the maximum
            // or the bias is not finite.
            auto move_up = [&](auto rises) {
                float pm[4];
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    pm[kb] = S[kb][0];
#pragma unroll
                    for (int i = 1; i < 16; ++i) pm[kb] = __builtin_fmaxf(pm[kb], S[kb][i]);
                }
                const float mx = max32(__builtin_fmaxf(__builtin_fmaxf(pm[0], pm[1]), __builtin_fmaxf(pm[2], pm[3])));
                if (last_key < T) v = 0.f;
                const double lev = (double)mx + (double)coef * (double)v;
                const float c = (float)(lev - R) + (mx + v) * 0.f;
                const bool move = rises(c, mx);
                if (DIRECT) nml = unseen ? 0.f : (c - mx) * LOG2E;
                if (__builtin_amdgcn_ballot_w64(move) != 0ull) {
                    asm volatile("" ::: "memory");
                    const float r = move ? __builtin_amdgcn_exp2f(-c * LOG2E) : 1.f;
                    R = move ? lev : R;
                    nml = move ? ((mx + v) * 0.f - mx) * LOG2E : nml;
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                        for (int i = 0; i < 16; ++i) O[cb][i] *= r;
#pragma unroll
                    for (int kb = 0; kb < 4; ++kb) l4[kb] *= r;
                }
            };
            if (DIRECT) {
                scores();
                move_up([&](float c, float) { return c > CMAX; });
                exponentials();
            } else {
                nml = 0.f;
                const float off = __builtin_fmaf(v, 0.f, (float)__builtin_fma((double)coef, (double)v, -R));
                if (!unseen) nml = off * LOG2E;
                unsigned long long high = ~0ull;
                if (__builtin_expect(j >= look_first.end, 1)) {
                    scores();
                    exponentials();
                    high = __builtin_amdgcn_ballot_w64(!(largest_of(Pf) <= PMAX));
                    if (high != 0ull) look_first.risen(j);
                }
                if (__builtin_expect(high != 0ull, 0)) {
                    asm volatile("" ::: "memory");
                    scores();                // there are no registers to keep them beside P
                    // as the row's own P shows it, which is rounded, so that it does not go by what its neighbours do
                    move_up([&](float, float mx) { return !unseen && !(p_of(mx, nml) <= PMAX); });
                    exponentials();
                }
            }
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int t2 = 0; t2 < 8; ++t2)
                    l4[kb] = add_pair(h2{Pf[2 * kb + (t2 >> 2)][2 * (t2 & 3)], Pf[2 * kb + (t2 >> 2)][2 * (t2 & 3) + 1]}, l4[kb]);
        }
        PASA_FENCE();
        __builtin_amdgcn_s_waitcnt(0x0F70 | CPW);        // this wavefront's share of V(j); that of K'(j + 1) may be on its way
        workgroup_barrier();
        PASA_FENCE();
        if (j < J_w) {
            const _Float16* lds_v = reinterpret_cast<const _Float16*>(smem + V_OFF);
            auto frag = [&](int n) { return *reinterpret_cast<const h8*>(lds_v + ((2 * (n / CB) + lh) * D + 32 * (n % CB) + lq) * 8); };
            h8 a[PF];
#pragma unroll
            for (int n = 0; n < PF; ++n) a[n] = frag(n);
            PASA_FENCE();
#pragma unroll
            for (int n = 0; n < 8 * CB; ++n) {
                O[n % CB] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[n % PF], Pf[n / CB], O[n % CB], 0, 0, 0);
                PASA_FENCE();
                if (n + PF < 8 * CB) a[n % PF] = frag(n + PF);
                PASA_FENCE();
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);          // no copy may be on its way into LDS when the workgroup ends
    if (qw0 >= Nq) return;
    const float l = sum32((l4[0] + l4[1]) + (l4[2] + l4[3]));
    if (part_o != nullptr) {
        const size_t rows_all = (size_t)(gridDim.x / (nqt * nsplit)) * Nq;
        const size_t grow = (size_t)split * rows_all + head * Nq + row;
        if (row_valid && lh == 0) {
            part_lr[grow * 2] = (double)l;
            part_lr[grow * 2 + 1] = l == l ? R : (double)l;
        }
        if (row_valid)
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int gq = 0; gq < 4; ++gq) {
                    const float4 v4 = {O[cb][4 * gq], O[cb][4 * gq + 1], O[cb][4 * gq + 2], O[cb][4 * gq + 3]};
                    *reinterpret_cast<float4*>(part_o + grow * D + 32 * cb + 8 * gq + 4 * lh) = v4;
                }
        return;
    }
    // through the buffer of the last K' tile: all wavefronts have read it, and the copy that went beyond it is in the other one
    const float oscale = 1.0f / l;
    store_rows<D, 1>(smem + ((J_wg - 1) & 1) * KT_BYTES + wave * (64 * D), [&](int, int cb, int i) { return O[cb][i] * oscale; },
                  o + (head * Nq + qw0) * D, Nq - qw0, lane, io_bf16);
}

template <bool CAUSAL, bool DIRECT>
hipError_t launch_fwd4(const PasaLaunch& p)
{
    constexpr int D = 64, LDS_BYTES = 3 * T * D * 2 + 4096;
    const int nqt = (p.Nq + 127) / 128, nsplit = p.nsplit < 1 ? 1 : p.nsplit;
    auto kern = pasa_fwd4<CAUSAL, DIRECT>;
    static std::atomic<unsigned long long> lds_limit_set{0ull};      // once per device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(lds_limit_set.load(std::memory_order_acquire) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        lds_limit_set.fetch_or(bit, std::memory_order_release);
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(nqt * p.Hq * p.B * nsplit)), dim3(256), LDS_BYTES, p.stream, (const _Float16*)p.q,
                       (const char*)p.ws, (_Float16*)p.o, (const _Float16*)p.kmean, p.Hq, p.Hkv, p.Nq, p.row0, p.N, nqt,
                       DIRECT ? p.scale : p.inva, p.io_bf16, p.gate,
                       nsplit, nsplit > 1 ? (float*)p.part_o : nullptr, nsplit > 1 ? (double*)p.part_lr : nullptr);
    e = hipGetLastError();
    if (e != hipSuccess || nsplit == 1) return e;
    return pasa_launch_merge(p.part_o, p.part_lr, p.o, (size_t)p.B * p.Hq * p.Nq, D, nsplit, p.io_bf16, nullptr, p.stream);
}

}  // namespace

hipError_t pasa_launch_fwd4(const PasaLaunch& p)
{
    if (p.variant == PASA_K_DIRECT) return p.causal ? launch_fwd4<true, true>(p) : launch_fwd4<false, true>(p);
    return p.causal ? launch_fwd4<true, false>(p) : launch_fwd4<false, false>(p);
}
