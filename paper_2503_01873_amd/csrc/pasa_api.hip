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
// each of its four wavefronts at least.  Not two where the rows of a KV head are one block and for S16 at d = 64 (`two` not set): 171 workgroups
// and more keep the memory busy alone, and a merge costs 5 us (a row
// each, in two pieces / whole: 24 sequences of 4000 keys, 8 KV heads, 75.0 / 68.1; 14 x 16 heads, d = 64, of 3000 / 12000 keys 28.8 / 25.6,
// 119.6 / 113.0; but 14 x 8 KV heads of 5000 keys in four pieces / whole 46.1 / 54.5); elsewhere the estimates decide (14 x 12 heads on 2, 5
// rows of 2301 keys in two pieces / whole 12.7 / 15.2).  Not up to 2048 keys, so that a row's result there does not depend on how many rows and
// sequences are given with it.  That is not where a split begins to pay: with the present merge kernel that is near 1400
// keys (1 row, 28 heads on 4, d = 128, us not split / split: 500 keys 6.2 / 9.7, 1000 keys 7.7 / 8.9, 1500 keys 9.8 / 9.1,
// 2047 keys 13.0 / 9.2; 4 sequences of 2047 keys 14.0 / 9.4).  Fewer than these, and two too, where the workspace ends: its last region is
// sized by wanted_splits (16 sequences of 1 row of 4999 keys get 4 of 8, 28 sequences of 5000 keys 2 of 4).
int rows_splits(int B, int Hkv, int G, int Nq, int rb, int N, int keys, bool two)
{
    const long groups = rows_workgroups(B, Hkv, G, Nq, rb), units = ((long)keys + 63) / 64;
    if (N <= 2048) return 1;
    long ns = 2 * kComputeUnits / groups;
    if (ns == 2 && !two) return 1;
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
// the fixed regions of the workspace hold), and the blocks of 16 rows per workgroup of pasa_rows, of rows per wavefront of HALVES.
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
// The factors of the estimates were fitted to 7400 calls of 128 to 32768 keys that ran on every kernel, as the kernels were before pasa_fwd
// took MFMAs of 16 x 16 x 32 and, with pasa_fwd4, exponentials without a maximum: the plan was 0.6 % behind the fastest kernel on average, 0.7 %
// S16.  With the kernels as they are it is 0.5 % behind on 203 prompts drawn like those (d = 128 0.6 %, S16 0.6 %, d = 64 0.4 %), four of them by a
// tenth to a sixth, and 6 % on 57 pieces, most of it in two that are planned as their whole.  The factors rank the kernels and are not
// times, above all at d = 64 and for the long launches of pasa_fwd, which take a tenth less.  Not all lie where these calls alone would put them:
// tests hold some calls to a kernel that is not their fastest (777 rows below, 8 heads, d = 64, of 2500 rows not causal), and calls near those go with
// them.  us, pasa_fwd / HALVES / pasa_rows, 28 heads on 4:
//   causal, 394 / 561 / 687 / 841 / 990 rows         15.3 / 11.7 / 9.1, 15.6 / 13.3 / 10.9, 20.2 / 15.0 / 18.4, 20.5 / 16.4 / 20.2, 25.2 / 18.4 / 22.6
//   causal, 1616 / 2089 / 2240 / 2813 / 4488 rows    36.8 / 29.7 / 41.9, 47.1 / 43.4 / 62.6, 52.9 / 46.1 / 68.9, 68.4 / 69.8 / 97.5, 134 / 153 / 223
//   not causal, 391 / 581 / 1006 / 2021 / 5746 rows  16.3 / 12.4 / 10.3, 18.6 / 13.9 / 18.5, 26.3 / 21.2 / 28.3, 54.0 / 64.0 / 86.6, 418 / 437 / 633
//   31 / 157 rows of 11699 / 9168 keys, 334 of 14242, 1206 of 22977    101 / 121 / 32.7, 179 / 98.9 / 58.6, 272 / 155 / 149, 448 / 565 / 591
//   S16, causal, 286 / 391 / 1792 / 3770 rows        10.9 / 10.9 / 7.6, 16.1 / 12.3 / 12.1, 46.0 / 34.8 / 84.6, 104 / 119 / 319
// planned on the fastest but for 687 (pasa_rows).  Pieces as the whole: 47 rows of 637 keys, not causal, 12.8 on HALVES, 6.6 on pasa_rows.
// d = 64, pasa_fwd / pasa_fwd4 / pasa_rows:
//   14 x 5 heads, not causal, 153 / 366 / 688 / 1162 rows     9.0 / 6.8 / 5.2, 11.2 / 8.5 / 11.9, 18.9 / 18.4 / 23.5, 49.2 / 39.7 / 52.9
//   14 x 5 heads, causal, 169 / 758 / 2321 / 10791 rows       8.1 / 6.7 / 5.6, 17.0 / 15.6 / 21.3, 81.0 / 74.3 / 109, 1346 / 1267 / 1676
//   one head, causal, 412 / 1664 / 18625 rows                 11.0 / 8.5 / 5.1, 25.3 / 21.5 / 6.8, 125 / 94.2 / 87.6
//   one head in one / two pieces on pasa_rows, causal, 5586 rows 25.3 / 19.5, not causal, 2536 / 3200 rows 10.1 / 13.0, 10.3 / 14.3
//   14 x 16 heads, 186 rows at the end of 8006 keys           154 / 166 / 195

// Equal workgroups, one to a compute unit, each `fixed` us and `steps` steps: of `alone` us, of `busy` where all compute units are at work
// (power), which takes part of the way with the square of the share that is.
double equal_rounds(double workgroups, double fixed, double alone, double busy, double steps)
{
    const double whole = floor(workgroups / kComputeUnits), rest = workgroups / kComputeUnits - whole;
    return whole * (fixed + busy * steps) + (rest > 0 ? fixed + (alone + (busy - alone) * rest * rest) * steps : 0.0);
}

// The longer of a chain and the work of the whole chip, and a tenth of the other
double longer(double chain, double work) { return chain > work ? chain + 0.1 * work : work + 0.1 * chain; }

// Causal, longest first: `most` steps in the longest workgroup, `mean` on average
double unequal_rounds(double workgroups, double fixed, double chain_step, double work_step, double most, double mean)
{
    return longer(fixed + chain_step * most, workgroups / kComputeUnits * (fixed + work_step * mean));
}

// pasa_rows, us of a key tile: the only workgroup of a compute unit; one of two or more, equal and causal; and of a pair's start and end
struct RowsStep {
    double alone, equal, causal, fixed;
};

// Two workgroups share a compute unit.  Equal ones come in rounds of 512 (32 heads, not causal, of 512 / 549 rows, 512 / 576 workgroups: 10.8 /
// 18.5 us).  Causal: the XCDs that share a list get ranges of unequal work (2 heads, d = 64, of 28830 rows: 558 us, evenly shared out
// it would be 357); a single list is dealt round.
double rows_time(const RowsStep& at, long workgroups, long lists, bool equal, double most, double mean)
{
    const double per = workgroups / (double)kComputeUnits;
    if (equal) {
        const double pair = at.fixed + 2 * at.equal * most, whole = floor(per / 2), rest = per - 2 * whole;
        return 4.0 + whole * pair + (rest == 0 ? 0.0 : rest <= 1 ? at.fixed / 2 + at.alone * most : pair);
    }
    const double uneven = lists > 1 && lists < 8 ? 1.584 - 0.073 * (double)lists : 1.0;
    return 4.0 + longer(at.alone * most, per * (at.fixed / 2 + at.causal * mean) * uneven);
}

// The merge kernel: its launch, and the partial outputs written and read again
double merge_us(int ns, size_t rows_all, int d) { return ns > 1 ? 5.5 + 2e-6 * (double)rows_all * ns * d : 0.0; }

// Pieces of a sequence whose keys are swept unsplit have the bits of the whole call: the kernels round P relative to different
// levels, so all pieces go to the kernel of the whole.  That holds for launches of at least kSplitBelow workgroups of 256 rows
// and for all up to 2048 keys; pieces start at multiples of 32 rows (rows of a wavefront stay together) and have 32 rows or
// more.  Shorter ones are decoding steps, which would lose five times (16 x 1 row of 4999 keys: 33 us, 173 on the
// kernel of the whole), except the end of a causal sequence of up to 2048 keys.  What it costs, us on the kernel of the whole /
// on the one that is fastest, 28 heads on 4, d = 128: 128 rows of 2048 keys 29.4 / 12.9, 512 rows 29.3 / 26.2, 32 rows of
// 1024 keys 16.2 / 7.8; 14 sequences, row 800 of 801 keys (every 32nd decoding step) 35.7 / 7.1.
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
    const bool one_block = (long)G * Nq <= 16, s16_64 = s16 && d == 64;
    if (may_split) r.nsplit = fitting(rows_splits(B, Hkv, G, Nq, r.row_blocks, N, most, !one_block && !s16_64), rows_all, d, room);
    if (one_block) return r;
    double rows_us;
    if (s16_64) {
        // a split has to save more than its merge costs
        if (r.nsplit > 1 && 0.85 * most_t * (r.nsplit - 1) < (rows_all > 1024 ? 8.0 : 6.0) * r.nsplit) r.nsplit = 1;
        const double uneven = !equal && B * Hq == 1 ? 1.3 : 1.0;
        const double work = 1.6 * uneven * rows_workgroups(B, Hkv, G, Nq, 2) * (5.5 / 512 + 0.52 / 256 * mean_t);
        const double alone = 0.85 * most_t / r.nsplit;
        rows_us = 4.0 + (work > alone ? work : alone) + (r.nsplit > 1 ? 6.0 : 0.0);
    } else {
        static const RowsStep steps[2][2] = {{{0.367, 0.2465, 0.35, 2.373}, {0.521, 0.3765, 0.4321, 3.166}},      // d = 64: 16 rows, 32
                                             {{0.713, 0.605, 0.6, 3}, {0.7579, 0.5543, 0.7044, 4.429}}};     // d = 128
        static const RowsStep steps_s16 = {0.83, 0.526, 1.0, 3.01};
        const int rb = s16 ? 1 : rows_blocks(B, Hkv, G, Nq);       // of the whole: pieces of it are to be planned as it is
        const RowsStep& at = s16 ? steps_s16 : steps[d == 128][rb - 1];
        const long workgroups = rows_workgroups(B, Hkv, G, Nq, rb), lists = (long)B * Hkv * (Nq < 16 ? 1 : G);
        auto us = [&](int ns) {
            const double t = rows_time(at, workgroups * ns, lists, equal, most_t / ns, mean_t / ns);
            // S16: weighed against the others, not a time, once there is more than a round of workgroups
            return (s16 && workgroups * ns > 2 * kComputeUnits ? 4.0 + 1.74 * (t - 4.0) : t) + merge_us(ns, rows_all, d);
        };
        rows_us = us(1);
        if (r.nsplit > 1) {
            const double split_us = us(r.nsplit);
            if (split_us < rows_us) rows_us = split_us;
            else r.nsplit = 1;
        }
    }
    if (d == 128) {
        const double most_h = ceil(ceil(most_t) / 2), mean_h = mean_t / 2 + 0.25, W = (double)B * Hq * ((Nq + 127) / 128);
        const double most_f = most_t / p.nsplit, mean_f = mean_t / p.nsplit;
        const double fwd_us = (equal ? equal_rounds(U * p.nsplit, 8.357, s16 ? 4.17 : 2.313, s16 ? 2.91 : 2.699, most_f)
                                     : unequal_rounds(U * p.nsplit, 8.357, s16 ? 2.51 : 2.111, s16 ? 3.17 : 2.76, most_f, mean_f)) * real +
                              merge_us(p.nsplit, rows_all, d);
        const double halves_us = equal ? equal_rounds(W, 8.34, s16 ? 3.69 : 2.45, s16 ? 3.52 : 2.935, most_h)
                                       : unequal_rounds(W, 8.34, s16 ? 2.78 : 2.2, s16 ? 3.15 : 2.738, most_h, mean_h);
        if (rows_us < 0.98 * (fwd_us < halves_us ? fwd_us : halves_us)) return r;
        // MFMAs of 32 rows where one round of workgroups leaves power to spare, because they are short or, causal, mostly shorter than the longest: there
        // instructions count (us, 32 rows / 16, one round, causal: 28 heads of 1024 rows 23.6 / 24.6, 12 heads of 2304 rows 37.7 / 39.4, 8 heads of 4000 rows
        // 67.0 / 68.4; 8 heads, not causal, 4096 rows 76.1 / 73.7; two rounds, causal: 28 heads of 2048 rows 49.6 / 47.7)
        if (halves_us < 0.98 * fwd_us) p = {Plan::HALVES, 1, W <= kComputeUnits && (most_h <= 4 || !equal) ? 1 : 2};
        return p;
    }
    // d = 64, S16: a step of pasa_fwd takes 2.0 to 2.55 us.  The others: of pasa_fwd 2.1 to 2.7, of pasa_fwd4 2.1 / 2.7 / 3.3 with one / two / three
    // workgroups on every compute unit, all of it a quarter longer than measured (see the line below).
    const double U_ns = U * p.nsplit, alone = (s16 ? 2.5 : 2.101) * most_t / p.nsplit, power = (real - 0.85) / 0.15;
    const double busy = s16 ? 2.0 + 0.55 * power : 2.14 + 0.55 * power;
    const double full = ((s16 ? causal != 0 : !equal) ? U_ns / 256 * mean_t
                         : U_ns <= 256 ? (0.75 + 0.25 * U_ns / 256) * most_t : ceil(U_ns / 256) * most_t) * busy / p.nsplit;
    const double longest = alone > full ? alone : full;
    if (s16) return rows_us <= 0.92 * (7.0 + longest + (p.nsplit > 1 ? 6.0 : 0.0)) ? r : p;
    const double fwd_us = 10.31 + longest + merge_us(p.nsplit, rows_all, d);
    Plan f = {Plan::FWD4, 1, 0};
    if (may_split) f.nsplit = fitting(fwd4_splits(B, Hq, Nq, N), rows_all, d, room);
    const double W = (double)B * Hq * ((Nq + 127) / 128) * f.nsplit, rest = fmod(W, 768.0);
    const double rounds = floor(W / 768) * 3.347 + (rest == 0 ? 0.0 : rest <= 256 ? 2.12 : rest <= 512 ? 2.711 : 3.347);
    const double alone4 = 2.12 * most_t, full4 = equal ? rounds * most_t : W / 768 * 3.347 * mean_t;
    const double fwd4_us = 8.423 + (alone4 > full4 ? alone4 : full4) / f.nsplit + merge_us(f.nsplit, rows_all, d);
    if (rows_us <= 0.7511 * (fwd_us < fwd4_us ? fwd_us : fwd4_us)) return r;
    return fwd4_us <= 1.005 * fwd_us ? f : p;
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

// For tests: the kernel of a call (bits 0 to 3) and its blocks of rows, -1 for none
int pasa_internal_plan(int variant, int counters, int B, int Hq, int Hkv, int Nq, int row0, int N, int d, int causal,
                       size_t workspace_bytes, int* nsplit)
{
    const size_t need = workspace_min_bytes(B, Hkv, N, d);
    if (check_shape(B, Hq, Hkv, N, d) != PASA_OK || workspace_bytes < need) return -1;
    const Plan p = plan_call(variant, counters != 0, true, B, Hq, Hkv, Nq, causal ? row0 : 0, N, d, causal, workspace_bytes - need);
    if (nsplit != nullptr) *nsplit = p.nsplit;
    return p.kernel | p.row_blocks << 4;
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
    p.halves = plan.kernel == Plan::HALVES ? plan.row_blocks : 0;
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
