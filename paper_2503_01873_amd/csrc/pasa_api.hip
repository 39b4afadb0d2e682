// libpasa host layer: the C ABI declared in include/pasa.h.
// Argument validation, the optimal-beta solve (host, fp64) and kernel dispatch.  No kernels here; the only device
// object is the fixed workspace of pasa_attn_fwd_static.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "pasa.h"
#include "pasa_device.h"
#include "pasa_kernels.h"

namespace {

constexpr int kShiftTile = 128;
constexpr int kMaxN = 262144;   // tile counters stay exactly representable in fp16 (STRICT16 statistics)

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; }

// Round x to a binary floating-point format with `prec` significand bits (including the hidden one),
// minimum normal exponent emin and maximum exponent emax (value < 2^(emax+1)); ties to even; gradual
// underflow; overflow to infinity.  fp16: (11, -14, 15).  bf16: (8, -126, 127).
double round_to_format(double x, int prec, int emin, int emax)
{
    if (x == 0.0 || isnan(x) || isinf(x)) return x;
    int e;
    frexp(x, &e);            // x = m * 2^e with 0.5 <= |m| < 1, so the leading bit has weight 2^(e-1)
    int lsb = e - prec;      // weight of the last kept bit
    if (lsb < emin - (prec - 1)) lsb = emin - (prec - 1);   // subnormal range: fixed spacing
    const double r = ldexp(nearbyint(ldexp(x, -lsb)), lsb); // nearbyint: ties to even in the default mode
    if (fabs(r) >= ldexp(1.0, emax + 1)) return copysign(INFINITY, x);
    return r;
}

double fl_tp(double x, int tp) { return tp == 0 ? round_to_format(x, 11, -14, 15) : round_to_format(x, 8, -126, 127); }

// The entries of the rounded shifting matrix of Appendix A: off-diagonal -b with b = fl(beta / n), diagonal
// a - b with a - b = fl(1 - beta / n) (Eq. (21)).  Both are step functions of beta.
struct RoundedPair {
    double a, b;
    bool operator==(const RoundedPair& o) const { return a == o.a && b == o.b; }
};

RoundedPair rounded_pair(double beta, int n, int tp)
{
    const double b = fl_tp(beta / n, tp);
    return {fl_tp(1.0 - beta / n, tp) + b, b};
}

// Eq. (20): the invariance that a*I - b*J really has, from its exact inverse (Theorem 2.1 with lambda = b / a).
double invariance_of_pair(const RoundedPair& p, int n)
{
    const double bn = p.b * n;
    return bn / (p.a * (p.a - bn)) + (1.0 - p.a) / p.a;
}

int check_shape(int B, int Hq, int Hkv, int N, int d)
{
    if (B <= 0 || Hq <= 0 || Hkv <= 0 || N <= 0 || d <= 0) return PASA_EINVAL;
    if (Hq % Hkv != 0) return PASA_EINVAL;
    if (d != 64 && d != 128) return PASA_EUNSUPPORTED;
    if (N > kMaxN) return PASA_EUNSUPPORTED;
    return PASA_OK;
}

}  // namespace

extern "C" {

const char* pasa_status_string(int status)
{
    switch (status) {
        case PASA_OK: return "ok";
        case PASA_EINVAL: return "invalid argument";
        case PASA_EUNSUPPORTED:
            return "unsupported size (d must be 64 or 128, N <= 262144, shift tile 128, N % 128 == 0 for the matrix shift)";
        case PASA_ELAUNCH: return "HIP runtime refused an allocation or a kernel launch";
        case PASA_EWORKSPACE: return "workspace missing, misaligned or too small";
        default: return "unknown status";
    }
}

int pasa_version(void) { return 100; }

double pasa_invariance_rounded(double beta, int n, int tp)
{
    if (!(beta >= 0.0) || !(beta < 1.0) || n <= 0 || (tp != 0 && tp != 1)) return NAN;
    return invariance_of_pair(rounded_pair(beta, n, tp), n);
}

double pasa_optimal_beta(double beta0, int n, int tp)
{
    if (!(beta0 > 0.0) || !(beta0 < 1.0) || n <= 0 || (tp != 0 && tp != 1)) return NAN;
    // The optimal accuracy condition beta / (1 - beta) = f(beta) (Eq. (16)) has a right-hand side that only depends on
    // the rounded pair (a, b), which is constant on intervals of beta.  On such an interval the condition is solved in
    // closed form, beta* = f / (1 + f); beta* is a solution iff it lies in the interval it was computed for, i.e. iff
    // rounding at beta* gives the same pair again.  Starting from the pair of beta0 and moving to the pair of the
    // candidate until it reproduces itself visits the same intervals as the iteration of Eq. (22) and ends exactly.
    RoundedPair pair = rounded_pair(beta0, n, tp);
    double beta = beta0;
    for (int visited = 0; visited < 256; ++visited) {
        const double f = invariance_of_pair(pair, n);
        beta = f / (1.0 + f);
        const RoundedPair again = rounded_pair(beta, n, tp);
        if (again == pair) return beta;
        pair = again;
    }
    return beta;     // no self-consistent interval found within the budget: the last candidate, as the iteration would give
}

}  // extern "C"

namespace {

// Workspace layout: the K'/V tiles, then (written by PASA_DIRECT's pre-processing) one fp16 shift vector of d halfs per
// tile in plain order, then (used by the adaptive entry point only) one 64-bit overflow counter per (batch, KV head),
// then one block of 32 x d halfs per 16 key tiles (PASA_MIXED: the tiles' mean keys; PASA_DIRECT: their shift vectors),
// then the region of the key split: per split and query row two doubles (sum, level) and the stored output (d floats).
size_t tiles_bytes(int B, int Hkv, int N, int d)
{
    const size_t ntile = ((size_t)N + kShiftTile - 1) / kShiftTile;      // a ragged last tile is padded
    return (size_t)4 * (size_t)B * (size_t)Hkv * ntile * kShiftTile * (size_t)d;
}

size_t k0_bytes(int B, int Hkv, int N, int d)
{
    const size_t ntile = ((size_t)N + kShiftTile - 1) / kShiftTile;
    const size_t raw = (size_t)2 * (size_t)B * (size_t)Hkv * ntile * (size_t)d;
    return (raw + 255) / 256 * 256;
}

size_t group_counter_bytes(int B, int Hkv)
{
    return ((size_t)8 * (size_t)B * (size_t)Hkv + 255) / 256 * 256;
}

size_t kmean_bytes(int B, int Hkv, int N, int d)
{
    const size_t ntile = ((size_t)N + kShiftTile - 1) / kShiftTile;
    return (size_t)B * (size_t)Hkv * ((ntile + 15) / 16) * 64 * (size_t)d;     // a multiple of 256
}

size_t kmean_offset(int B, int Hkv, int N, int d)
{
    return tiles_bytes(B, Hkv, N, d) + k0_bytes(B, Hkv, N, d) + group_counter_bytes(B, Hkv);
}

// Everything but the key-split region: what a call needs at least.
size_t workspace_min_bytes(int B, int Hkv, int N, int d)
{
    return kmean_offset(B, Hkv, N, d) + kmean_bytes(B, Hkv, N, d);
}

// Key split.  A launch of fewer than 192 workgroups (256 query rows of one head each) leaves compute units idle; then
// the key tiles of every workgroup are divided among up to 256 / workgroups of them, in pieces of 16 tiles, at most 16.
constexpr int kComputeUnits = 256;      // MI355X
constexpr int kSplitBelow = 192;
constexpr int kMaxSplit = 16;
constexpr size_t kSplitFloorBytes = (size_t)1 << 20;   // always there, so that short query chunks (decoding) can split

int wanted_splits(int B, int Hq, int Nq, int N)
{
    const long units = ((long)Nq + 255) / 256 * Hq * B;
    const int nblk16 = (int)((((long)N + kShiftTile - 1) / kShiftTile + 15) / 16);
    if (units >= kSplitBelow || nblk16 < 2) return 1;
    long ns = kComputeUnits / units;
    if (ns > nblk16) ns = nblk16;
    if (ns > kMaxSplit) ns = kMaxSplit;
    return ns < 2 ? 1 : (int)ns;
}

// Workgroups of pasa_rows with `rb` blocks of 16 rows, without a key split: the rows of a KV head's query heads are one
// list when fewer than 16 are given, one list per query head otherwise.
long rows_workgroups(int B, int Hkv, int G, int Nq, int rb)
{
    const int R = 16 * rb;
    return (long)B * Hkv * (Nq < 16 ? ((long)G * Nq + R - 1) / R : (long)G * ((Nq + R - 1) / R));
}

// Blocks of 16 rows per workgroup.  One while that gives a workgroup to every compute unit at most: 28 heads on 4, d = 128,
// 32767 keys, us with one / two blocks: 127 rows (224 workgroups of one) 146 / 187, 255 rows 276 / 190.
int rows_blocks(int B, int Hkv, int G, int Nq)
{
    return (long)G * Nq <= 16 || rows_workgroups(B, Hkv, G, Nq, 1) <= kComputeUnits ? 1 : 2;
}

// Workgroups that share the keys of a row block: as many as make two to a compute unit, each with a unit of 64 keys for
// each of its four wavefronts at least.  Not two: 171 workgroups and more keep the memory busy alone, and a merge costs 5 us (a row
// each, in two pieces / whole: 24 sequences of 4000 keys, 8 KV heads, 75.0 / 68.1; 14 x 16 heads, d = 64, of 3000 / 12000 keys 28.8 / 25.6,
// 119.6 / 113.0; but 14 x 8 KV heads of 5000 keys in four pieces / whole 46.1 / 54.5).  Not up to 2048 keys, so that a row's result there does not depend on how many rows and
// sequences are given with it.  That is not where a split begins to pay: with the present merge kernel that is near 1400
// keys (1 row, 28 heads on 4, d = 128, us not split / split: 500 keys 6.2 / 9.7, 1000 keys 7.7 / 8.9, 1500 keys 9.8 / 9.1,
// 2047 keys 13.0 / 9.2; 4 sequences of 2047 keys 14.0 / 9.4).  Fewer than these where the workspace ends: its last region is sized by
// wanted_splits (16 sequences of 1 row of 4999 keys get 4 of 8).
int rows_splits(int B, int Hkv, int G, int Nq, int rb, int N, int keys)
{
    const long groups = rows_workgroups(B, Hkv, G, Nq, rb), units = ((long)keys + 63) / 64;
    if (N <= 2048) return 1;
    long ns = 2 * kComputeUnits / groups;
    if (ns == 2) return 1;
    if (ns > (units + 3) / 4) ns = (units + 3) / 4;
    return ns < 1 ? 1 : (int)ns;
}

// pasa_fwd4: as many workgroups as are resident at once (three to a compute unit), pieces of 8 tiles at least.  Not up to
// 2048 keys, for the same reason (a split would be two pieces of one).
int fwd4_splits(int B, int Hq, int Nq, int N)
{
    const long units = ((long)Nq + 127) / 128 * Hq * B, pieces = ((long)N + 1023) / 1024;
    if (N <= 2048) return 1;
    long ns = 3 * kComputeUnits / units;
    if (ns > pieces) ns = pieces;
    return ns < 1 ? 1 : ns > kMaxSplit ? kMaxSplit : (int)ns;
}

size_t split_row_bytes(int d) { return (size_t)d * 4 + 16; }

// The kernel of a call, in how many pieces its keys are swept (as many as the kernel's rule wants and the `room` bytes behind
// the fixed regions of the workspace hold), and the blocks of 16 rows per workgroup of pasa_rows.
struct Plan {
    enum { FWD, HALVES, FWD4, ROWS } kernel;
    int nsplit, row_blocks;
};

int fitting(int ns, size_t rows_all, int d, size_t room)
{
    while (ns > 1 && (size_t)ns * rows_all * split_row_bytes(d) > room) --ns;
    return ns;
}

// pasa_fwd (256 rows of one head per workgroup) takes every call.  Without counters, at d = 128 and not for the variants whose
// state has no merge (STRICT16) or that only serve comparison (NAIVE16), it can run as workgroups of 128 rows whose two
// groups of wavefronts take the even and the odd key tiles (HALVES).  MIXED, DIRECT and S16 without
// counters can also go to pasa_rows (16 or 32 query rows, the keys shared out among the wavefronts), MIXED and DIRECT at
// d = 64 to pasa_fwd4 (128 rows of one head, four wavefronts).  pasa_rows takes every call whose rows of a KV head fit one block (a decoding step reads its keys
// once and not once per query head); otherwise the estimate below, from measured rates, says which is fastest.
//
// 28 heads on 4, d = 128, us of pasa_fwd / HALVES / pasa_rows.  Causal prompts of 512 / 1024 / 2048 / 3000 rows: 20.2 / 16.1 / 11.0,
// 29.7 / 21.7 / 25.6, 50.7 / 45.9 / 71, 81 / 88 / -.  128 / 512 / 1024 rows at the end of 16384 keys: 262 / 174 / 75, 309 / 174 / 164, 310 /
// 234 / 323.  8 heads of 3000 / 4096 rows, not causal: 60.5 (split) / 48.0 / 54.9, 80.0 (split) / 72.8 / 94.8.
// 14 sequences, 1 / 20 / 64 rows of 6000 keys, pasa_fwd / pasa_rows: 189 / 34, 189 / 65, 192 / 124.
// S16, 28 heads on 4, pasa_fwd / pasa_rows: 1 row of 500 / 6000 / 16000 keys 15.8 / 6.4, 43.9 / 10.6, 47.9 / 12.4; 128 rows 17.3 / 7.7,
// 114 / 40.1, 290 / 96.8; 16 heads, d = 64, 500 rows of 3000 keys 65.6 / 24.3.
// d = 128, causal, pasa_fwd / HALVES / pasa_rows: 28 heads of 614 / 768 / 1035 / 2196 rows 16.0 / 13.6 / 15.1, 20.6 / 15.0 / 16.8, 25.5 / 19.4 /
// 23.9, 52.9 / 45.1 / 66.2 (of these only 1035 is planned on the fastest); 12 heads on 2 of 2185 rows 47.6 / 30.2 / 35.7; 4 x 8 heads of
// 651 rows 20.1 / 14.5 / 16.1.
// The factors of the estimates are fitted to 220 such calls of 150 to 6000 keys (on average 0.2 % behind the fastest kernel), so they rank the kernels and are not times: 14 x 5 heads of 9216 rows,
// d = 64, not causal, are put at 1843 us (pasa_fwd) and 1793 (pasa_fwd4) and take 1630 and 1490; a call whose estimates lie within
// a few per cent may go to the slower kernel.
// d = 64, pasa_fwd / pasa_fwd4 / pasa_rows: 16 heads, causal, of 2290 rows 38 / 31 / 24 (stays on pasa_fwd4); 2 x 16 heads of 508 rows 14.3 / 9.5 / 7.5; 14 x 5 heads,
// causal, of 168 / 221 rows 8.6 / 6.9 / 5.5, 8.6 / 6.7 / 5.4; 14 x 28 heads on 4 of 198 rows 17 / 13.6 / 21.  The factors are fitted to 240 such calls
// (2.1 % behind the fastest kernel on average before, 0.9 now).
// d = 64, pasa_fwd / pasa_fwd4: 14 x 5 heads of 1000 / 2000 / 4000 rows, not causal, 50.7 / 34.8, 134 / 103, 420 / 356, causal
// 26.5 / 24.1, 70 / 60, 224 / 206; 2 x 16 heads of 4000 rows, not causal (a round and a third of pasa_fwd4) 174 / 184;
// one head of 16384 rows, causal, both split: 79 / 67, and 101 with pasa_rows.

// Equal workgroups, `slots` of them at once, each `fixed` us and `tiles` steps of 2.5 us -- 2.8 when all compute units
// are busy (power; sustained it is 3.5, for both kernels alike), which takes part of the way with the square of the share that is.
double equal_rounds(double workgroups, double slots, double fixed, double tiles)
{
    const double whole = floor(workgroups / slots), rest = (workgroups - whole * slots) / slots;
    return whole * (fixed + 2.8 * tiles) + (rest > 0 ? fixed + (2.5 + 0.3 * rest * rest) * tiles : 0.0);
}

// Causal: `most` steps in the longest workgroup and `mean` on average, longest first.
double unequal_rounds(double workgroups, double slots, double fixed, double most, double mean)
{
    const double chain = fixed + 2.23 * most, work = workgroups / slots * (fixed + 3.41 * mean);
    return chain > work ? chain + 0.1 * work : work + 0.1 * chain;
}

// Pieces of a sequence whose keys are swept unsplit have the bits of the whole call: the kernels round P relative to different
// levels, so all pieces go to the kernel of the whole.  That holds for launches of at least kSplitBelow workgroups of 256 rows
// and for all up to 2048 keys; pieces start at multiples of 32 rows (rows of a wavefront stay together) and have 32 rows or
// more.  Shorter ones are decoding steps, which would lose five times (16 x 1 row of 4999 keys: 33 us, 173 on the
// kernel of the whole), except the end of a causal sequence of up to 2048 keys.  What it costs, us on the kernel of the whole /
// on the one that is fastest, 28 heads on 4, d = 128: 128 rows of 2048 keys 31.6 / 13.8, 512 rows 31.6 / 26.7, 32 rows of
// 1024 keys 19.4 / 8.6; 14 sequences, row 800 of 801 keys (every 32nd decoding step) 40 / 9.
bool keeps_the_bits_of_the_whole(int B, int Hq, int Nq, int row0, int N, int causal)
{
    if (wanted_splits(B, Hq, Nq, N) > 1 || (causal && row0 % 32 != 0)) return false;
    return Nq >= 32 || (causal && N <= 2048 && row0 + Nq >= N);
}

Plan plan_call(int variant, bool counters, bool may_split, int B, int Hq, int Hkv, int Nq, int row0, int N, int d, int causal,
               size_t room)
{
    const int rows_given = Nq;
    if (keeps_the_bits_of_the_whole(B, Hq, Nq, row0, N, causal)) {
        may_split = false;
        Nq = N;
        row0 = 0;
    }
    const size_t rows_all = (size_t)B * Hq * Nq;
    const double merge = 6.0;      // us: its launch and 4 us for few rows, 8 for many
    Plan p = {Plan::FWD, 1, 0};
    if (may_split && variant != PASA_STRICT16) p.nsplit = fitting(wanted_splits(B, Hq, Nq, N), rows_all, d, room);
    if (counters || variant == PASA_STRICT16 || variant == PASA_NAIVE16) return p;
    const bool s16 = variant == PASA_S16;      // its pseudo-average costs pasa_rows a second pass over the keys; blocks of 16 rows only

    // keys that the last row sees, and that a row sees on average; in tiles
    const int most = causal && row0 < N - Nq ? row0 + Nq : N, mean = causal && row0 < N - Nq / 2 ? row0 + Nq / 2 : N;
    const double most_t = most / (double)kShiftTile, mean_t = mean / (double)kShiftTile;
    const bool equal = mean_t > 0.8 * most_t;
    const double U = (double)B * Hq * ((Nq + 255) / 256), real = Nq < 256 ? 0.85 + 0.15 * Nq / 256.0 : 1.0;

    const int G = Hq / Hkv;
    Plan r = {Plan::ROWS, 1, s16 ? 1 : rows_blocks(B, Hkv, G, rows_given)};
    double rows_us;
    {
        if (may_split) r.nsplit = fitting(rows_splits(B, Hkv, G, Nq, r.row_blocks, N, most), rows_all, d, room);
        if ((long)G * Nq <= 16) return r;
        // a split has to save more than its merge costs (d = 64, one head of 2275 rows: 10.1 us in two pieces, 8.7 whole; of 2812 rows,
        // not causal, 13.0 / 10.6)
        if (r.nsplit > 1 && (s16 ? 0.85 : 0.55) * most_t * (r.nsplit - 1) < (rows_all > 1024 ? merge + 2.0 : merge) * r.nsplit) r.nsplit = 1;
        const double uneven = !equal && B * Hq == 1 ? 1.3 : 1.0;     // one causal head: no even ranges for the XCDs
        // us of a step: d = 128, causal, less beyond 1024 keys, where the longest blocks come first; d = 64, not much less where the
        // other kernels would split their keys
        const bool others_split = wanted_splits(B, Hq, Nq, N) > 1 || fwd4_splits(B, Hq, Nq, N) > 1;
        const double step = d == 64 ? (s16 ? 0.52 : others_split ? 0.54 : 0.44) : causal && N > 1024 ? 0.71 : 0.845;
        const double work = (!s16 ? 1.0 : d == 64 ? 1.6 : 2.6) * uneven * rows_workgroups(B, Hkv, G, Nq, 2) * (5.5 / 512 + step / 256 * mean_t);
        const double alone = (s16 ? 0.85 : 0.55) * most_t / r.nsplit;
        rows_us = 4.0 + (work > alone ? work : alone) + (r.nsplit > 1 ? merge : 0.0);
    }
    if (d == 128) {
        const double most_h = ceil(ceil(most_t) / 2), mean_h = mean_t / 2 + 0.25, W = (double)B * Hq * ((Nq + 127) / 128);
        const double fwd_us = (equal ? equal_rounds(U * p.nsplit, 256, 9.4, most_t / p.nsplit)
                                     : unequal_rounds(U * p.nsplit, 256, 9.4, most_t / p.nsplit, mean_t / p.nsplit)) * real +
                              (p.nsplit > 1 ? merge : 0.0);
        const double halves_us = equal ? equal_rounds(W, 256, 10.5, most_h) : unequal_rounds(W, 256, 10.5, most_h, mean_h);
        if (rows_us < 0.98 * (fwd_us < halves_us ? fwd_us : halves_us)) return r;
        if (halves_us < 0.98 * fwd_us) p = {Plan::HALVES, 1, 0};
        return p;
    }
    // d = 64: a step of pasa_fwd takes 2.0 to 2.55 us, one of pasa_fwd4 1.73 / 2.44 / 3.17 with one / two / three workgroups on every
    // compute unit (3.7 sustained, under the power limit)
    const double U_ns = U * p.nsplit, alone = (s16 ? 2.5 : 2.0) * most_t / p.nsplit;
    const double full = (causal ? U_ns / 256 * mean_t : U_ns <= 256 ? (0.75 + 0.25 * U_ns / 256) * most_t : ceil(U_ns / 256) * most_t) *
                        (2.0 + 0.55 * (real - 0.85) / 0.15) / p.nsplit;
    const double fwd_us = (s16 ? 7.0 : 8.1) + (alone > full ? alone : full) + (p.nsplit > 1 ? merge : 0.0);
    Plan f = {Plan::FWD4, 1, 0};
    if (may_split) f.nsplit = fitting(fwd4_splits(B, Hq, Nq, N), rows_all, d, room);
    const double W = (double)B * Hq * ((Nq + 127) / 128) * f.nsplit, rest = fmod(W, 768.0);
    const double rounds = floor(W / 768) * 3.17 + (rest == 0 ? 0.0 : rest <= 256 ? 1.73 : rest <= 512 ? 2.44 : 3.17);
    const double alone4 = 1.73 * most_t, full4 = causal ? W / 768 * 3.17 * mean_t : rounds * most_t;
    const double fwd4_us = 7.6 + (alone4 > full4 ? alone4 : full4) / f.nsplit + (f.nsplit > 1 ? merge : 0.0);
    if (rows_us <= (s16 ? 0.92 : 0.95) * (s16 || fwd_us < fwd4_us ? fwd_us : fwd4_us)) return r;
    return !s16 && fwd4_us <= 0.98 * fwd_us ? f : p;
}

size_t split_region_bytes(int B, int Hq, int N, int d)
{
    const int ns = wanted_splits(B, Hq, N, N);
    size_t need = ns > 1 ? (size_t)ns * (size_t)B * Hq * N * split_row_bytes(d) : 0;
    if (need < kSplitFloorBytes) need = kSplitFloorBytes;
    return (need + 255) / 256 * 256;
}

}  // namespace

extern "C" {

size_t pasa_attn_fwd_workspace(int B, int Hq, int Hkv, int N, int d)
{
    if (check_shape(B, Hq, Hkv, N, d) != PASA_OK) return 0;
    return workspace_min_bytes(B, Hkv, N, d) + split_region_bytes(B, Hq, N, d);
}

size_t pasa_attn_fwd_workspace_min(int B, int Hkv, int N, int d)
{
    if (check_shape(B, Hkv, Hkv, N, d) != PASA_OK) return 0;
    return workspace_min_bytes(B, Hkv, N, d);
}

int pasa_internal_plan(int variant, int counters, int B, int Hq, int Hkv, int Nq, int row0, int N, int d, int causal,
                       size_t workspace_bytes, int* nsplit)
{
    const size_t need = workspace_min_bytes(B, Hkv, N, d);
    if (check_shape(B, Hq, Hkv, N, d) != PASA_OK || workspace_bytes < need) return -1;
    const Plan p = plan_call(variant, counters != 0, true, B, Hq, Hkv, Nq, causal ? row0 : 0, N, d, causal, workspace_bytes - need);
    if (nsplit != nullptr) *nsplit = p.nsplit;
    return p.kernel;
}

unsigned pasa_internal_quotient(unsigned n, unsigned d) { return fast_div(d).quotient(n); }

}  // extern "C"

namespace {

// Entries of the shifting matrix M = I/alpha - beta J/(alpha T) of Eq. (10), alpha = 1/kscale, each rounded to
// fp16: a on the diagonal, b elsewhere.  The pre-processing kernel takes a - b and b.
void rounded_shift_matrix(double beta, double kscale, double* a_minus_b, double* b)
{
    const double alpha = 1.0 / kscale;
    const double off = beta / (alpha * (double)kShiftTile);
    const double a16 = round_to_format(1.0 / alpha - off, 11, -14, 15);
    const double b16 = round_to_format(0.0 - off, 11, -14, 15);
    *a_minus_b = a16 - b16;    // exact: both are fp16 values
    *b = b16;
}

int shift_keys_common(const void* k, void* kprime, int B, int Hkv, int N, int d, double beta, double kscale,
                      int shift_mode, void* k0out, void* stream)
{
    const int st = check_shape(B, Hkv, Hkv, N, d);
    if (st != PASA_OK) return st;
    if (k == nullptr || kprime == nullptr || !aligned(k, 16) || !aligned(kprime, 16) || k == kprime) return PASA_EINVAL;
    if (!(beta >= 0.0) || !(beta < 1.0) || !isfinite(kscale) || !(kscale > 0.0)) return PASA_EINVAL;
    double c1 = beta, c2 = kscale;
    if (shift_mode == PASA_PREP_MATRIX) {
        if (N % kShiftTile != 0) return PASA_EUNSUPPORTED;   // M is a full 128 x 128 matrix
        rounded_shift_matrix(beta, kscale, &c1, &c2);
    }
    if (shift_mode == PASA_PREP_DIRECT && (k0out == nullptr || !aligned(k0out, 16) || k0out == kprime || k0out == k))
        return PASA_EINVAL;
    const hipError_t e = pasa_launch_prep(k, nullptr, nullptr, kprime, B, Hkv, N, d, c1, c2, shift_mode, 0, k0out,
                                          nullptr, nullptr, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? PASA_OK : PASA_ELAUNCH;
}

}  // namespace

extern "C" {

int pasa_shift_keys(const void* k, void* kprime, int B, int Hkv, int N, int d, double beta, double kscale, void* stream)
{
    return shift_keys_common(k, kprime, B, Hkv, N, d, beta, kscale, PASA_PREP_MEAN, nullptr, stream);
}

int pasa_shift_keys_matrix(const void* k, void* kprime, int B, int Hkv, int N, int d, double beta, double kscale,
                           void* stream)
{
    return shift_keys_common(k, kprime, B, Hkv, N, d, beta, kscale, PASA_PREP_MATRIX, nullptr, stream);
}

int pasa_shift_keys_matrix_mfma(const void* k, void* kprime, int B, int Hkv, int N, int d, double beta, double kscale,
                                void* stream)
{
    const int st = check_shape(B, Hkv, Hkv, N, d);
    if (st != PASA_OK) return st;
    if (k == nullptr || kprime == nullptr || !aligned(k, 16) || !aligned(kprime, 16) || k == kprime) return PASA_EINVAL;
    if (!(beta >= 0.0) || !(beta < 1.0) || !isfinite(kscale) || !(kscale > 0.0)) return PASA_EINVAL;
    if (N % kShiftTile != 0) return PASA_EUNSUPPORTED;
    double amb, b16;
    rounded_shift_matrix(beta, kscale, &amb, &b16);
    const hipError_t e = pasa_launch_shift_gemm(k, nullptr, kprime, B, Hkv, N, d, amb + b16, b16, 0, nullptr,
                                                static_cast<hipStream_t>(stream));
    return e == hipSuccess ? PASA_OK : PASA_ELAUNCH;
}

int pasa_shift_keys_direct(const void* k, void* kprime, void* k0, int B, int Hkv, int N, int d, double beta, double kscale,
                           void* stream)
{
    return shift_keys_common(k, kprime, B, Hkv, N, d, beta, kscale, PASA_PREP_DIRECT, k0, stream);
}

namespace {

// Resolved numeric parameters of one call.
struct Params {
    int variant;
    double beta;      // shift fraction used by the pre-processing kernel (matrix mode: a - b)
    double kscale;    // factor folded into K' (matrix mode: b)
    int matrix_mode;  // K' by the fp16-rounded shifting matrix instead of by the tile mean
    int mfma_shift;   // ... and that product on the matrix core (fp32 accumulation) instead of exactly
    int io_bf16;      // q, k, v, o hold bf16
    float inva;       // beta/(1-beta) rounded to the statistics precision
    unsigned long long* overflow_s;
    unsigned long long* nonfinite_o;
    const unsigned long long* gate;   // set by the adaptive entry point only
};

int resolve(const pasa_opts* opts, float scale, Params* out)
{
    if (!isfinite(scale) || !(scale > 0.f)) return PASA_EINVAL;
    pasa_opts op = {-1.f, PASA_MIXED, kShiftTile, nullptr, nullptr, PASA_SHIFT_MEAN, PASA_IO_F16};
    if (opts != nullptr) op = *opts;
    if (op.variant < PASA_MIXED || op.variant > PASA_DIRECT) return PASA_EINVAL;
    if (op.shift_mode != PASA_SHIFT_MEAN && op.shift_mode != PASA_SHIFT_MATRIX && op.shift_mode != PASA_SHIFT_MATRIX_MFMA)
        return PASA_EINVAL;
    if (op.variant == PASA_DIRECT && op.shift_mode != PASA_SHIFT_MEAN) return PASA_EINVAL;   // it has its own shift
    if (op.io_dtype != PASA_IO_F16 && op.io_dtype != PASA_IO_BF16) return PASA_EINVAL;
    if (op.shift_tile != 0 && op.shift_tile != kShiftTile) return PASA_EUNSUPPORTED;
    if (!(op.beta < 1.f)) return PASA_EINVAL;              // also rejects NaN
    // beta and the invariance beta/(1-beta) in fp64.  Default by mean: the invariance is exactly 63.5.  Default by
    // matrix: the paper's adopted solution of the optimal accuracy condition for fp16 and n = 128 (Table 3).
    const double beta_default = op.shift_mode != PASA_SHIFT_MEAN ? 0.984497 : 63.5 / 64.5;
    double beta = op.beta < 0.f ? beta_default : (double)op.beta;
    double kscale = (double)scale;
    if (op.variant == PASA_NAIVE16) {   // no shift, static scaling applied after the first GEMM (Eq. (1), (2))
        beta = 0.0;
        kscale = 1.0;
    }
    const double inva_d = beta / (1.0 - beta);
    out->variant = op.variant;
    out->beta = beta;
    out->kscale = kscale;
    out->io_bf16 = op.io_dtype == PASA_IO_BF16;
    out->matrix_mode = op.shift_mode != PASA_SHIFT_MEAN && op.variant != PASA_NAIVE16;
    out->mfma_shift = out->matrix_mode && op.shift_mode == PASA_SHIFT_MATRIX_MFMA;
    if (out->matrix_mode) rounded_shift_matrix(beta, kscale, &out->beta, &out->kscale);
    out->inva = op.variant == PASA_STRICT16 ? (float)round_to_format(inva_d, 11, -14, 15) : (float)inva_d;
    out->overflow_s = op.overflow_s;
    out->nonfinite_o = op.nonfinite_o;
    out->gate = nullptr;
    return PASA_OK;
}

int check_workspace(const void* ws, size_t bytes, size_t need)
{
    return (ws == nullptr || !aligned(ws, 256) || bytes < need) ? PASA_EWORKSPACE : PASA_OK;
}

}  // namespace

}  // extern "C"

namespace {

int prepare_kv_impl(const void* k, const void* v, int B, int Hkv, int N, int d, float scale, const pasa_opts* opts,
                    void* workspace, size_t workspace_bytes, void* stream, const unsigned long long* gate)
{
    if (k == nullptr || v == nullptr || !aligned(k, 16) || !aligned(v, 16)) return PASA_EINVAL;
    Params pr;
    int st = resolve(opts, scale, &pr);
    if (st != PASA_OK) return st;
    pr.gate = gate;
    st = check_shape(B, Hkv, Hkv, N, d);
    if (st != PASA_OK) return st;
    if (pr.matrix_mode && N % kShiftTile != 0) return PASA_EUNSUPPORTED;   // M is a full 128 x 128 matrix
    const size_t need = workspace_min_bytes(B, Hkv, N, d);
    st = check_workspace(workspace, workspace_bytes, need);
    if (st != PASA_OK) return st;
    const int mode = pr.variant == PASA_DIRECT ? PASA_PREP_DIRECT : pr.matrix_mode ? PASA_PREP_MATRIX : PASA_PREP_MEAN;
    void* k0out = static_cast<char*>(workspace) + tiles_bytes(B, Hkv, N, d);
    void* kmean = (pr.variant == PASA_MIXED || pr.variant == PASA_DIRECT)
                      ? static_cast<char*>(workspace) + kmean_offset(B, Hkv, N, d) : nullptr;
    if (pr.mfma_shift) {
        // V by the re-tiling blocks of the pre-processing kernel, K' by the GEMM (pr.beta carries a - b, pr.kscale b)
        hipError_t e2 = pasa_launch_prep(nullptr, v, workspace, nullptr, B, Hkv, N, d, 0.0, 1.0, PASA_PREP_MEAN, pr.io_bf16,
                                         nullptr, nullptr, pr.gate, static_cast<hipStream_t>(stream));
        if (e2 == hipSuccess)
            e2 = pasa_launch_shift_gemm(k, workspace, nullptr, B, Hkv, N, d, pr.beta + pr.kscale, pr.kscale, pr.io_bf16,
                                        kmean, static_cast<hipStream_t>(stream));
        return e2 == hipSuccess ? PASA_OK : PASA_ELAUNCH;
    }
    const hipError_t e = pasa_launch_prep(k, v, workspace, nullptr, B, Hkv, N, d, pr.beta, pr.kscale, mode, pr.io_bf16,
                                          k0out, kmean, pr.gate, static_cast<hipStream_t>(stream));
    return e == hipSuccess ? PASA_OK : PASA_ELAUNCH;
}

}  // namespace

extern "C" {

int pasa_prepare_kv(const void* k, const void* v, int B, int Hkv, int N, int d, float scale, const pasa_opts* opts,
                    void* workspace, size_t workspace_bytes, void* stream)
{
    return prepare_kv_impl(k, v, B, Hkv, N, d, scale, opts, workspace, workspace_bytes, stream, nullptr);
}

int pasa_attn_fwd_prepared(const void* q, void* o, int B, int Hq, int Hkv, int N, int d, int causal, float scale,
                           const pasa_opts* opts, void* workspace, size_t workspace_bytes, void* stream)
{
    return pasa_attn_fwd_chunk(q, o, B, Hq, Hkv, N, 0, N, d, causal, scale, opts, workspace, workspace_bytes, stream);
}

}  // extern "C"

namespace {

int fwd_chunk_impl(const void* q, void* o, int B, int Hq, int Hkv, int Nq, int row0, int N, int d, int causal,
                   float scale, const pasa_opts* opts, void* workspace, size_t workspace_bytes, void* stream,
                   unsigned long long* overflow_group, const unsigned long long* gate)
{
    if (q == nullptr || o == nullptr || !aligned(q, 16) || !aligned(o, 16) || o == q) return PASA_EINVAL;
    if (causal != 0 && causal != 1) return PASA_EINVAL;
    if (Nq <= 0 || row0 < 0) return PASA_EINVAL;
    Params pr;
    int st = resolve(opts, scale, &pr);
    if (st != PASA_OK) return st;
    st = check_shape(B, Hq, Hkv, N, d);
    if (st != PASA_OK) return st;
    if (Nq > kMaxN || row0 > kMaxN) return PASA_EUNSUPPORTED;
    if (pr.matrix_mode && N % kShiftTile != 0) return PASA_EUNSUPPORTED;
    const size_t need = workspace_min_bytes(B, Hkv, N, d);
    st = check_workspace(workspace, workspace_bytes, need);
    if (st != PASA_OK) return st;
    PasaLaunch p;
    p.q = q; p.ws = workspace; p.o = o;
    p.kmean = static_cast<const char*>(workspace) + kmean_offset(B, Hkv, N, d);
    p.B = B; p.Hq = Hq; p.Hkv = Hkv; p.N = N; p.d = d;
    p.Nq = Nq; p.row0 = causal ? row0 : 0;
    p.causal = causal;
    p.variant = pr.variant;
    p.io_bf16 = pr.io_bf16;
    p.inva = pr.inva;
    p.scale = scale;
    p.overflow_s = pr.overflow_s;
    p.nonfinite_o = pr.nonfinite_o;
    p.overflow_group = overflow_group;
    p.gate = gate;
    // key split: as many ways as the rule wants and the bytes behind the fixed regions hold
    const size_t rows_all = (size_t)B * Hq * Nq;
    const bool counters = overflow_group != nullptr || pr.overflow_s != nullptr || pr.nonfinite_o != nullptr;
    const Plan plan = plan_call(pr.variant, counters, gate == nullptr, B, Hq, Hkv, Nq, p.row0, N, d, causal, workspace_bytes - need);
    const int ns = plan.nsplit;
    p.nsplit = ns;
    p.halves = plan.kernel == Plan::HALVES;
    char* split_base = static_cast<char*>(workspace) + need;
    p.part_lr = split_base;                                              // [ns][rows][2] doubles
    p.part_o = split_base + (size_t)ns * rows_all * 16;                  // [ns][rows][d] floats
    p.stream = static_cast<hipStream_t>(stream);
    const hipError_t e = plan.kernel == Plan::ROWS ? pasa_launch_rows(p, plan.row_blocks)
                         : plan.kernel == Plan::FWD4 ? pasa_launch_fwd4(p) : pasa_launch_fwd(p);
    return e == hipSuccess ? PASA_OK : PASA_ELAUNCH;
}

}  // namespace

extern "C" {

int pasa_attn_fwd_chunk(const void* q, void* o, int B, int Hq, int Hkv, int Nq, int row0, int N, int d, int causal,
                        float scale, const pasa_opts* opts, void* workspace, size_t workspace_bytes, void* stream)
{
    return fwd_chunk_impl(q, o, B, Hq, Hkv, Nq, row0, N, d, causal, scale, opts, workspace, workspace_bytes, stream,
                          nullptr, nullptr);
}

int pasa_attn_fwd_adaptive(const void* q, const void* k, const void* v, void* o, int B, int Hq, int Hkv, int N, int d,
                           int causal, float scale, const pasa_opts* opts, void* workspace, size_t workspace_bytes,
                           void* stream)
{
    // every check of both passes first, so that nothing is enqueued on error
    if (q == nullptr || k == nullptr || v == nullptr || o == nullptr) return PASA_EINVAL;
    if (!aligned(q, 16) || !aligned(k, 16) || !aligned(v, 16) || !aligned(o, 16)) return PASA_EINVAL;
    if (o == q || o == k || o == v) return PASA_EINVAL;
    if (causal != 0 && causal != 1) return PASA_EINVAL;
    if (opts == nullptr || opts->overflow_s == nullptr || !aligned(opts->overflow_s, 8)) return PASA_EINVAL;
    if (opts->nonfinite_o != nullptr || opts->variant == PASA_NAIVE16) return PASA_EINVAL;
    if (opts->shift_mode == PASA_SHIFT_MATRIX_MFMA) return PASA_EINVAL;    // the GEMM pre-pass has no per-head gate
    Params pr;
    int st = resolve(opts, scale, &pr);
    if (st != PASA_OK) return st;
    st = check_shape(B, Hq, Hkv, N, d);
    if (st != PASA_OK) return st;
    if (pr.matrix_mode && N % kShiftTile != 0) return PASA_EUNSUPPORTED;
    st = check_workspace(workspace, workspace_bytes, workspace_min_bytes(B, Hkv, N, d));
    if (st != PASA_OK) return st;
    // the per-(batch, KV head) counters live behind the tiles and the shift vectors; cleared by a small kernel
    unsigned long long* group_cnt = reinterpret_cast<unsigned long long*>(
        static_cast<char*>(workspace) + tiles_bytes(B, Hkv, N, d) + k0_bytes(B, Hkv, N, d));
    if (pasa_launch_zero(group_cnt, B * Hkv, static_cast<hipStream_t>(stream)) != hipSuccess) return PASA_ELAUNCH;
    // pass 1: no shift, raw scores rounded to fp16, counting those that leave the fp16 range -- in total (the
    // caller's counter) and per (batch, KV head)
    pasa_opts first = *opts;
    first.variant = PASA_NAIVE16;
    first.shift_mode = PASA_SHIFT_MEAN;
    first.beta = -1.f;
    st = prepare_kv_impl(k, v, B, Hkv, N, d, scale, &first, workspace, workspace_bytes, stream, nullptr);
    if (st != PASA_OK) return st;
    st = fwd_chunk_impl(q, o, B, Hq, Hkv, N, 0, N, d, causal, scale, &first, workspace, workspace_bytes, stream,
                        group_cnt, nullptr);
    if (st != PASA_OK) return st;
    // pass 2: the caller's variant; the workgroups of a (batch, KV head) whose counter is zero leave at once, so its
    // query heads keep the result of pass 1
    pasa_opts second = *opts;
    second.overflow_s = nullptr;
    st = prepare_kv_impl(k, v, B, Hkv, N, d, scale, &second, workspace, workspace_bytes, stream, group_cnt);
    if (st != PASA_OK) return st;
    return fwd_chunk_impl(q, o, B, Hq, Hkv, N, 0, N, d, causal, scale, &second, workspace, workspace_bytes, stream,
                          nullptr, group_cnt);
}

int pasa_attn_fwd_ex(const void* q, const void* k, const void* v, void* o, int B, int Hq, int Hkv, int N, int d,
                     int causal, float scale, const pasa_opts* opts, void* workspace, size_t workspace_bytes,
                     void* stream)
{
    // all checks of both halves first, so that nothing is enqueued on error
    if (q == nullptr || k == nullptr || v == nullptr || o == nullptr) return PASA_EINVAL;
    if (!aligned(q, 16) || !aligned(k, 16) || !aligned(v, 16) || !aligned(o, 16)) return PASA_EINVAL;
    if (o == q || o == k || o == v) return PASA_EINVAL;
    if (causal != 0 && causal != 1) return PASA_EINVAL;
    Params pr;
    int st = resolve(opts, scale, &pr);
    if (st != PASA_OK) return st;
    st = check_shape(B, Hq, Hkv, N, d);
    if (st != PASA_OK) return st;
    if (pr.matrix_mode && N % kShiftTile != 0) return PASA_EUNSUPPORTED;
    st = check_workspace(workspace, workspace_bytes, workspace_min_bytes(B, Hkv, N, d));
    if (st != PASA_OK) return st;
    st = pasa_prepare_kv(k, v, B, Hkv, N, d, scale, opts, workspace, workspace_bytes, stream);
    if (st != PASA_OK) return st;
    return pasa_attn_fwd_prepared(q, o, B, Hq, Hkv, N, d, causal, scale, opts, workspace, workspace_bytes, stream);
}

int pasa_attn_fwd(const void* q, const void* k, const void* v, void* o, int B, int Hq, int Hkv, int N, int d,
                  int causal, float scale, void* stream)
{
    // validate before allocating anything: run the checks of the _ex entry point against a dummy workspace size
    const int st = check_shape(B, Hq, Hkv, N, d);
    if (q == nullptr || k == nullptr || v == nullptr || o == nullptr) return PASA_EINVAL;
    if (st != PASA_OK) return st;
    const size_t need = pasa_attn_fwd_workspace(B, Hq, Hkv, N, d);
    hipStream_t s = static_cast<hipStream_t>(stream);
    void* ws = nullptr;
    if (hipMallocAsync(&ws, need, s) != hipSuccess || ws == nullptr) {
        (void)hipGetLastError();
        return PASA_ELAUNCH;
    }
    const int rc = pasa_attn_fwd_ex(q, k, v, o, B, Hq, Hkv, N, d, causal, scale, nullptr, ws, need, stream);
    if (hipFreeAsync(ws, s) != hipSuccess) {
        (void)hipGetLastError();
        return rc == PASA_OK ? PASA_ELAUNCH : rc;
    }
    return rc;
}

}  // extern "C"

// ---------------------------------------------------------------------------------------------
// The entry point that allocates nothing.  Its workspace (shifted keys, re-tiled values, shift vectors) is this
// fixed array in device memory; every GPU the library is used on holds its own copy at its own address until the
// process ends.  In host code the array's name only stands for the symbol: the address on the current device comes
// from hipGetSymbolAddress, once per device, and only that address is handed to the kernels.
// ---------------------------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[PASA_STATIC_WORKSPACE_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU, filled on the first call there

int static_scratch(void** out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return PASA_ELAUNCH;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
            (void)hipGetLastError();
            return PASA_ELAUNCH;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return PASA_OK;
}

}  // namespace

extern "C" int pasa_attn_fwd_static(const void* q, const void* k, const void* v, void* o, int B, int Hq, int Hkv, int N,
                                    int d, int causal, float scale, const pasa_opts* opts, void* stream)
{
    const int st = check_shape(B, Hq, Hkv, N, d);
    if (st != PASA_OK) return st;
    // sizes beyond the fixed array are refused before anything else is looked at; what the fixed regions leave of the
    // array serves the key split
    const size_t need = workspace_min_bytes(B, Hkv, N, d);
    if (need == 0 || need > (size_t)PASA_STATIC_WORKSPACE_BYTES) return PASA_EWORKSPACE;
    void* ws = nullptr;
    const int sp = static_scratch(&ws);
    if (sp != PASA_OK) return sp;
    // every byte of the workspace that the main kernel reads is rewritten by the pre-processing kernel of the same
    // call (the padding keys of a ragged last tile included), so nothing has to be cleared between calls
    return pasa_attn_fwd_ex(q, k, v, o, B, Hq, Hkv, N, d, causal, scale, opts, ws, (size_t)PASA_STATIC_WORKSPACE_BYTES,
                            stream);
}
