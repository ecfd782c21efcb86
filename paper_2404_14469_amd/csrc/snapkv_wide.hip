// Window scoring and voting in two streaming passes for prompts whose KV heads are met by many window
// rows (Listing 1: the compute_attn call and the column sum; Eq. 1): grouped-query heads and wide windows.
//
// The single-read kernel (snapkv_fused.hip) keeps every exponential in registers until its row's normaliser
// is known, so a wave holds 32 rows x 64 keys, a KV head with 128 window rows is cut into four parts, every part
// streams the head's keys through the compute units again, and two thirds of the vector instructions go to the
// row maxima, hand-offs and votes of only 64 keys.  Here nothing is kept: all rows of a block meet every key
// of a round while it is on chip, first for the row statistics (wide_stats), then, once these are merged, for
// the votes (wide_votes).  K is read from memory once per pass whatever the number of query heads, and a logit
// costs a multiply-add, an exponential and an addition (or a multiply-add) per pass.
//
//   * The window rows of a KV head form blocks of whole query heads, at most eight 16-row units each, or four where the
//     KV head has no more (RUW); a unit of work is one block.  A wave owns 32 of the block's rows, its Q in registers as
//     MFMA fragments.
//   * The keys of a unit are cut into at most 64 slices of RPS rounds of 128 keys, into up to 256 if the prompt has
//     fewer than four units, or into fewer so that all slices of more than eight units find a place at once.  The
//     slice length depends on the prompt's length and its own heads alone, so a head's result does not depend on which
//     other layers or prompts share the launch.
//   * A round's keys pass through LDS (landing registers -> two buffers, one barrier a round), where four groups
//     of waves x two parts of the keys (blocks of 64 rows: two groups x four parts) read them as fragments; the next round is on
//     its way meanwhile.
//   * A single prompt (or the only one of a batch that comes here) whose slices all find a place at once has both passes in one launch (wide_once).
//   * Otherwise a persistent grid of two workgroups per compute unit walks the slices of all units (of all prompts or layers of
//     the call) in order, a contiguous run of whole slices each (of the votes: of rounds); a launch of one prompt whose slices all find a place at
//     once has a workgroup per slice.
//
// What bounds it: the stream of keys, and arithmetic that does not hide behind it.  32 layers of 32/8 heads of 31337 keys take
// 406 + 480 us (one session differs from another by about ten of each).  What follows was measured when the statistics took their logits rows x
// keys, in a session with 414 + 481 (back to back 430 + 492; the single-read kernel 1218): the same loops without the arithmetic 384 + 471, with keys
// that are always in the cache 334 + 351, and the keys alone 337 at 6.1 TB/s.  The votes' pass also stores 131 MB.  Counters of the present
// kernels (profiles/sq_counters_gqa_two_pass.txt, 32768 keys): of the 778 thousand cycles of wide_stats a SIMD's matrix unit is busy
// for 263 and its vector instructions take 385 (rows x keys: 436); of the 960 of wide_votes 262 and 444.  Tried on the way: all 128 rows in one
// wave with Q in LDS (two waves per SIMD, 425 + 512 us, and 240 registers); keys brought to LDS without registers, a ring of four
// rounds of 64 keys (456 + 522); a second set of landing registers (spills).  At 131072 keys, W = 64 (two blocks per
// head): 97 + 103 us against 277 us.
//
// The row reference.  Exponentials are taken relative to a reference of the row that is known before its keys are: its
// largest logit among the prompt's first four keys (sixteen where a block has 64 rows).  The argument s - ref is rounded
// to fp32, so the terms that matter must not lie far from the reference: a round in which a row's logits exceed it by about 2^kRaiseAt raises the row's
// reference to its largest logit less kRaiseBelow for the rest of the slice and takes its exponentials again, and
// wide_votes uses the largest of the slices' references.  Normally distributed logits get there at 4.5 standard
// deviations where one is 4.6 (base two), and not at all where it is 2.6.  No sum can overflow.  The margin below
// the largest logit keeps the many small terms of a peaked row nearer to the reference.  Relative error of the votes
// against float64 (2-norm, 1e-8; 18461 keys, 32/8 heads, 32 rows), single-read kernel / a reference that stays at the
// first key's logit / as it is: logits N(0, 1.8 nats) 12.2 / 12.6 / 12.3; with 40 keys 6, 20 and 40 nats above those
// 12.1 / 11.9 / 10.6, 15.8 / 17.5 / 15.2 and 28.1 / 34.5 / 28.0.  Checking and raising cost 0.8 of 64 us per call at
// 28471 keys, 0.5 of 67 at 32749 and nothing measurable at 131072.
//
// The row's origin (blocks of 64 rows).  Most of the error is that of the logits themselves, whose partial sums are rounded four
// times on the way.  Here they do not start from zero but from minus the row's origin: the first sixteen keys' logits fall into
// four quads, and the second largest of the quads' maxima is the origin (the largest may be a first token that every row attends
// to).  The sums of the logits that matter then end nearer to zero.  Reference, maxima and exponents are all counted from the
// origin, so nothing else changes; wide_stats leaves it behind a unit's slices.  It costs no time (262144 keys, 32/8 heads, W = 16 251 us
// a call with it and without).  Error of votes within a factor of two of the 1024th largest (2-norm of the relative errors, 1e-8, 32
// heads), logits N(0, s nats) and clusters, the single-read kernel (and from 262145 keys on or with W = 64: its front and rest) / the
// two passes without / with the origin, s = 0.45, 0.9, 1.8 and 3.6:
//   W = 16, four query heads, 140001 keys: 4.5 / 4.4 / 4.4, 5.6 / 5.4 / 5.2, 14.1 / 14.1 / 10.1 and 52.6 / 52.9 / 30.4;
//     380000 keys: 29.6 / 4.5 / 4.5, 28.5 / 5.7 / 5.5, 35.1 / 15.9 / 11.5 and 77.7 / 57.3 / 34.2;
//   W = 64, one query head, 140001 keys: 25.6 / 4.6 / 4.6, 26.5 / 5.3 / 5.1, 22.7 / 8.6 / 6.9 and 51.4 / 35.9 / 21.4.
// With the first key 8, 20 and 40 nats above the rest (W = 16, s = 1.8): 14.7 / 14.7 / 10.1, 41 / 41 / 31 and 206 / 205 / 140.  Started
// from minus the reference instead: 0.61 to 0.71 of the first figure without such a key, but 1.2 to 1.8 of it with one.
//
// wide_stats takes its logits keys x rows (the operands exchanged): a lane has four keys of one row instead of one key of four rows, so
// that it keeps two references and two sums instead of eight of each, and the sums over keys need an exchange between lanes only
// once a slice, over four lanes instead of sixteen.  118 registers instead of 127, and microseconds per call, rows x keys / keys x rows: 28471
// keys, 32/8 heads 56.85 / 56.39; 32749 token-major 59.33 / 58.47; 131072, W = 64 217.0 / 215.8 (two runs of one
// side differ by 0.1 to 0.3 %); the pass of 32 layers of 31337 keys, both in turn in one session, 409 (404 to 417) / 406 (403 to 411): no more than its runs differ.  The registers it frees are not enough for a second set of landing registers (14 to 18 spilled, 44.1 -> 48.0
// for the two passes at 28471 keys); both rows' products piece by piece, for two chains of MFMAs and fewer registers of keys, change nothing.
// The error of votes near the selection's threshold against float64 is what it was: over fifteen of the shapes and spreads named above
// 0.999 of it on average, 0.988 to 1.008 singly.  wide_votes, which sums over rows, stays with rows x keys.
//
// MFMA layout: that of snapkv_fused.hip (16x16x32, lane l: row / column l % 16, contraction slice l / 16;
// accumulator register r is row (l / 16) * 4 + r, column l % 16; the 16-byte pieces 4p + l / 16 of a row).
#include "snapkv_internal.h"
#include "snapkv_handoff.h"
#include "snapkv_help.h"
#include "snapkv_shares.h"

#include <algorithm>
#include <type_traits>

namespace snapkv {

__device__ unsigned g_wide_timeouts = 0;   // workgroups of wide_once that reached the bound on their turns (none does, see there)

bool reset_wide_timeouts() {
    const unsigned zero = 0;
    return hipMemcpyToSymbol(HIP_SYMBOL(g_wide_timeouts), &zero, sizeof zero) == hipSuccess;
}
unsigned read_wide_timeouts() {
    unsigned v = 0;
    if (hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_wide_timeouts), sizeof v) != hipSuccess) return ~0u;
    return v;
}

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 wbf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 wf16x8;
typedef __attribute__((ext_vector_type(4))) float wf32x4;

struct w_bf16 {};
struct w_f16 {};

constexpr int kWaves = 8;                    // waves per workgroup, two workgroups per compute unit
constexpr int kThreads = kWaves * 64;
constexpr int kRound = kWaves * 16;          // keys of a round: every wave brings one 16-key tile to LDS
constexpr int kSlices = 64;                  // slices per unit at most,
constexpr int64_t kPlaces = 256;             //   or as many as give a prompt of few units this many in all,
constexpr int64_t kPlacesAll = 512;          //   or a prompt of many, up to kMaxOnce, no more than this in all: the places of a chip
constexpr int64_t kMaxOnce = 32;             //   of 256 compute units (a fixed number, so that results do not depend on the device)
constexpr int kWaveRows = 2;                 // 16-row units of a wave
constexpr float kRaiseAt = 0x1p16f;          // exponential (of a lane's sum) from which a row's reference is raised,
constexpr float kRaiseMin = 8.f;             //   by rows whose largest logit lies this far above it (base two),
constexpr float kRaiseBelow = 7.f;           //   to that logit less this
// Window rows of a KV head (in whole 16-row units) times keys from which the two passes beat the single-read kernel.
// Microseconds per call, 32/8 heads of 128 in bf16, this path / the single-read kernel, one layer and four in one call:
//   W = 32 (128 rows):  8192 keys 51 / 45, 71 / 73;  16384: 57 / 55, 93 / 105;  20000: 60 / 70, 110 / 167;
//                      40001: 75 / 108, 194 / 323;  131072: 141 / 182, 483 / 632
//   W = 64 (256 rows):  8192: 57 / 53, 91 / 104;  10007: 65 / 73, 100 / 169;  28471: 85 / 110, 189 / 320;
//                      131072: 206 / 314, 785 / 1167
// Few KV heads (W = 32, single-read kernel / 64 slices per unit / kPlaces in all):
//   1 head: 18439 keys 40 / 41 / 39;  46087: 45 / 50 / 43;  131072: 55 / 80 / 53;  700001: 313 / 292 / 116
//   2 heads: 27655: 46 / 46 / 42;  131072: 77 / 85 / 66;  32 layers of 1 head, 31337: 196 / 144 / 151
// (with 512 in all: 1 head, 46087: 55, 131072: 67; 2 heads, 27655: 52)
// Where one launch does it, the line lies lower the more units a prompt has.  Single-read kernel / this path:
//   1 and 2 units of 128 rows: 14000 keys 29 / 30, -;  16384: 28 / 31, 29 / 32;  18000: 30 / 32, 34 / 33
//   4 units: 11000: 34 / 37;  14000: 34.3 / 32.4;  16384: 34.5 / 32.8;  18000: 43 / 35
//   8 units: 8192: 40 / 42;  14000: 43.9 / 41.2;  16384: 44.0 / 42.0;  18000: 59 / 45;  two layers: 14000: 60.5 / 63.5;  16384: 60.7 / 59.0;  four:
//            14000: 95 / 85;  18000: 157 / 94;  three: 16384: 78 / 82 (as many keys as that kernel takes in one go)
//   12 units: 12300: 58 / 50;  16 units: 12300: 66 / 53;  of 256 rows a KV head 6200: 50.7 / 45.1, two layers 67.8 / 65.5, three 86 / 74;
//   32 units: 12300: 101 / 66;  16384: 101 / 72;  two layers 12300: 173 / 121
// More than kMaxOnce units, which have the two launches, gain from the same line where a KV head has 128 rows, where it has 256 but for 8192 keys, and
// in layers; with 512 rows and slices of one round (no more than 8192 keys) some single prompts lose a little:
//   128 rows: 33 units: 12300: 99 / 79;  16384: 98 / 87;  40: 12300: 111 / 87;  16384: 112 / 104;  64: 12300: 164 / 118;  16384: 170 / 144;  two layers of 40:
//            12300: 224 / 144;  16384: 226 / 205;  three of 33: 14000: 286 / 217
//   256 rows: 34 units: 6200: 66 / 62;  8192: 66 / 63;  40: 6200: 71 / 66;  7680: 75 / 65;  8192: 70 / 75;  48: 6200: 79 / 71;  8192: 79 / 82;  56: 8192: 86 / 88;
//            64: 6200: 95 / 79;  8192: 94 / 80;  two layers of 40: 6200: 142 / 91;  8192: 142 / 107
//   512 rows: 36 units: 3100: 50 / 50;  3600: 52 / 55;  4096: 52 / 53;  4590: 67 / 53;  48: 3600: 56 / 59;  4096: 57 / 63;  64: 3600: 65 / 65;  4096: 65 / 58;
//            two layers of 36: 4096: 104 / 68
// Few layers from four units on, between these lines and 9 << 18: 4 units: two of 16400 keys 62 / 52, three of 18400 78 / 58;  8 units: two of 16400 99 / 67,
// three 138 / 79;  12 units: two of 12300 84 / 72, three of 18000 194 / 104;  16 units of 256 rows: two of 6200 90 / 60, four 181 / 80.
// Prompts of a batch between these lines and 9 << 18, which shared a joint launch before, mostly gain too, and lose where they are few among shorter ones
// (compress_batch in snapkv_api.hip has the figures).
constexpr int64_t min_row_keys(int64_t units) { return units > 8 ? 3 << 19 : units >= 4 ? (1 << 21) + 1 : 9 << 18; }
// With 64 rows the single-read kernel is faster by 12 to 28 % up to 131072 keys, but for lengths that leave it compute units idle
// (W = 16, 32/8 heads, this path / that kernel: 16384 keys 43 / 34, 40001: 61 / 62, 65536: 80 / 67, 90001: 98 / 103, 131072: 125 / 112;
// W = 64, 32 heads, 32768: 125 / 103, 131072: 443 / 374).  Beyond that it has W = 16 with one row unit a part, the four parts of a KV head
// one after another, up to 262144 keys, and everything else, as W = 16 from 262145 keys on, as a front read once and a rest that the
// streaming kernel reads twice.  Microseconds per call, this path / those:
//   W = 16, 32/8 heads:  131073 keys 128 / 274;  140001: 150 / 283;  175001: 185 / 287;  262144: 250 / 348;  380000: 356 / 509
//   W = 64, 32/32 heads: 131073: 463 / 758;  140001: 502 / 782;  175001: 603 / 827;  262144: 848 / 1177;  300001: 981 / 1390
//   one KV head, W = 16 and 64: 132000: 45 / 58, 48 / 75;  1000001: 144 / 268, 149 / 328
// A window of two row units and two query heads a KV head: W = 32, 32/16 heads
//   131073: 249 / 239;  150001: 285 / 273;  160001: 298 / 290;  170001: 313 / 344;  262144: 440 / 589;
// the line is that of sixteen KV heads, though with four of them this path is the faster one from 131073 keys on (76 / 95; 170001: 89 / 120).
// Windows of 49 to 63 rows and one query head do not fall into blocks of 32 rows, and the single-read kernel holds 65536 keys of them; from there
// to 131072 they go as front and rest too (not measured against this path).
constexpr int64_t kMinRowKeys64 = (1 << 23) + 64, kMinRowKeys64of2 = 5 << 21;
constexpr int64_t kMaxRounds = 1 << 26;      // rounds of one prompt at most (kMaxWide of them are counted in 32 bits)

template <int D> struct KFrag {
    static constexpr int NP = D / 32;        // 16-byte pieces per lane and row (2-byte elements)
    uint4 v[NP];
};

__device__ __forceinline__ wf32x4 mma16(w_bf16, uint4 a, uint4 b, wf32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(wbf16x8, a), __builtin_bit_cast(wbf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ wf32x4 mma16(w_f16, uint4 a, uint4 b, wf32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(wf16x8, a), __builtin_bit_cast(wf16x8, b), c, 0, 0, 0);
}
template <typename T, int D>
__device__ __forceinline__ wf32x4 logits16(const KFrag<D>& q, const KFrag<D>& k, wf32x4 acc = {0.f, 0.f, 0.f, 0.f}) {
#pragma unroll
    for (int p = 0; p < KFrag<D>::NP; ++p) acc = mma16(T{}, q.v[p], k.v[p], acc);
    return acc;
}

// Blocks of 64 rows: logits are counted from an origin of the row (see "The row reference").
template <int RUW> constexpr bool kOrigin = RUW == 4;
template <int RUW> constexpr int kExtra = kOrigin<RUW> ? 1 : 0;
template <int RUW> struct Origins {
    wf32x4 neg[kOrigin<RUW> ? kWaveRows : 1];
    template <typename T, int D> __device__ __forceinline__ wf32x4 logits(const KFrag<D>& q, const KFrag<D>& k, int i) const {
        if constexpr (kOrigin<RUW>) return logits16<T, D>(q, k, neg[i]);
        else return logits16<T, D>(q, k);
    }
};

// Sums and maxima over the lanes of other rows of sixteen: exchanges between the wave's halves and between the two rows of a half.
struct Two {
    float a, b;
};
__device__ __forceinline__ Two swap32(float a, float b) {
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return {__uint_as_float(x[0]), __uint_as_float(x[1])};
}
__device__ __forceinline__ Two swap16(float a, float b) {
    const auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return {__uint_as_float(x[0]), __uint_as_float(x[1])};
}
__device__ __forceinline__ float halves(float a, float b) {   // lanes 0-31: a of lane l and l + 32, lanes 32-63: b
    const Two x = swap32(a, b);
    return x.a + x.b;
}
__device__ __forceinline__ float quarters(float a, float b) {   // even rows of 16 lanes: a of both rows of the half, odd ones: b
    const Two x = swap16(a, b);
    return x.a + x.b;
}
__device__ __forceinline__ float rows_max(float x) {          // over the four rows of sixteen lanes
    const Two y = swap32(x, x);
    x = fmaxf(y.a, y.b);
    const Two z = swap16(x, x);
    return fmaxf(z.a, z.b);
}

// Orders LDS traffic only: the K rounds in flight are not waited for.
__device__ __forceinline__ void lds_meet() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One prompt (or layer) of a launch.
struct WideEntry {
    const char* q;
    const char* k;
    float* vote;
    float2* part;        // [units][NS + kExtra][RUW * 16] per slice and row: (reference, sum of 2^(s - reference));
                         //   behind a unit's slices, RUW = 4: (-origin, 0) per row
    int64_t k_hs;        // bytes between the K rows of consecutive KV heads
    int64_t vpitch;      // floats between vote rows
    unsigned round_begin; // rounds of the entries before this one
    int L, n, RPS, NS, units;
};
template <int N> struct WideArgs {   // N: 1 or kMaxWide (a single prompt's launch has little to fetch before its first load)
    int count, direct, g, W, UH, hb, nblk;   // hb query heads per block, nblk blocks per KV head, UH row units per query head
    int inv_uh;                      // 256 / UH rounded up: a row unit's query head is ru * inv_uh >> 8
    float c2;
    int64_t k_rs;
    const int32_t* table;            // paged K (one entry only): see ScoreGeom
    int page;
    int64_t pages, row0;
    unsigned rounds;                 // of all entries: each workgroup's share is share rounds, one more for the first `more`
    unsigned share, more;
    bool reversed;                   // the statistics' shares are handed out as share_of says
    unsigned spin_limit;             // wide_once: polls before a workgroup helps itself,
    unsigned* gave_up;               //   and null, or a word that is set when one gives up
    unsigned* zeros;                 // words the selection expects to be zero (see WideClear); null: none
    int64_t nzeros;
    unsigned* flag;
    WideEntry e[N];
};

// Where a workgroup stands in the launch's sequence of rounds (all wave-uniform).
struct Cursor {
    int e, kv, blk, sl, rd;          // entry, KV head and block of the unit, slice of the unit, round of the slice
    int L, n, RPS, NS, units;
    const char* kb;                  // K rows of the unit's head
};

template <int N> __device__ __forceinline__ void enter(const WideArgs<N>& A, Cursor& c) {
    const WideEntry& E = A.e[c.e];
    c.L = E.L;
    c.n = E.n;
    c.RPS = E.RPS;
    c.NS = E.NS;
    c.units = E.units;
    c.kb = E.k + (int64_t)c.kv * E.k_hs;
}

// Where the statistics of the cursor's unit begin.
template <int RUW, int N> __device__ __forceinline__ int64_t unit_part(const WideArgs<N>& A, const Cursor& c) {
    return ((int64_t)c.kv * A.nblk + c.blk) * (c.NS + kExtra<RUW>) * (RUW * 16);
}

// First round at or after `r` at which a slice begins.
template <int N> __device__ __forceinline__ unsigned slice_start(const WideArgs<N>& A, unsigned r) {
    if (r >= A.rounds) return A.rounds;
    int e = 0;
    if constexpr (N > 1)
        for (int i = 1; i < A.count; ++i)
            if (r >= A.e[i].round_begin) e = i;
    return A.e[e].round_begin + whole_slices(r - A.e[e].round_begin, (unsigned)A.e[e].RPS);
}
// Where the workgroup's stretch of rounds begins.  The statistics are of whole slices (WHOLE); the votes, which take a row's weight as it is
// wherever they begin, are shared out by rounds.  With whole slices in both passes, of which a workgroup of a few layers' launch has two
// or three, a part of the chip had nothing to do at the end.  Microseconds per call, W = 64, 32/8 heads: 3 layers of 8500 keys 78.1 / 76.3, of 12300
// 101.1 / 96.2, of 17000 115.7 / 112.5;  4 of 10500 103.5 / 100.3, of 15000 114.5 / 111.3, of 32000 207 / 208;  W = 32: 4 of 28000 138.5 / 134.2, 32 of
// 31337 1004 / 1005.
template <bool WHOLE, int N> __device__ __forceinline__ unsigned share(const WideArgs<N>& A, unsigned wg) {
    const unsigned r = begin_rounds(A.share, A.more, wg);
    return WHOLE ? slice_start(A, r) : r;
}

template <int N> __device__ __forceinline__ Cursor cursor_at(const WideArgs<N>& A, unsigned r) {
    Cursor c;
    c.e = 0;
    if constexpr (N > 1)
        for (int i = 1; i < A.count; ++i)
            if (r >= A.e[i].round_begin) c.e = i;
    const WideEntry& E = A.e[c.e];
    const unsigned in = r - E.round_begin, slice = in / (unsigned)E.RPS;
    const int u = (int)(slice / (unsigned)E.NS);
    c.sl = (int)(slice % (unsigned)E.NS);
    c.kv = u / A.nblk;
    c.blk = u % A.nblk;
    c.rd = (int)(in % (unsigned)E.RPS);
    enter(A, c);
    return c;
}

// Where the workgroup starts and how many rounds are its own.  A launch whose slices all find a place at once has a
// workgroup per slice (grid: slices of a unit x blocks of a KV head x KV heads; no divisions before the first load).
template <bool WHOLE, int N> __device__ __forceinline__ Cursor begin_share(const WideArgs<N>& A, int& rounds) {
    if (N == 1 && A.direct) {
        Cursor c;
        c.e = 0;
        c.kv = (int)blockIdx.z;
        c.blk = (int)blockIdx.y;
        c.sl = (int)blockIdx.x;
        c.rd = 0;
        enter(A, c);
        rounds = c.RPS;
        return c;
    }
    const unsigned own = WHOLE ? share_of(blockIdx.x, gridDim.x, A.reversed) : blockIdx.x;
    const unsigned r0 = share<WHOLE>(A, own), r1 = share<WHOLE>(A, own + 1);
    rounds = (int)(r1 - r0);
    return cursor_at(A, r0 < A.rounds ? r0 : 0u);
}

// The next round; stays on the launch's last one.  Returns whether the unit changed.
template <int N> __device__ __forceinline__ bool advance(const WideArgs<N>& A, Cursor& c) {
    if (++c.rd < c.RPS) return false;
    if (c.sl + 1 < c.NS) {
        ++c.sl;
        c.rd = 0;
        return false;
    }
    if (c.blk + 1 < A.nblk) {
        ++c.blk;
    } else if ((c.kv + 1) * A.nblk < c.units) {
        ++c.kv;
        c.blk = 0;
    } else if (N > 1 && c.e + 1 < A.count) {
        ++c.e;
        c.kv = c.blk = 0;
    } else {
        --c.rd;
        return false;
    }
    c.sl = c.rd = 0;
    enter(A, c);
    return true;
}

// The workgroup's waves, lanes and K stream; shared by both passes.
template <typename T, int D, bool PAGED, int N, int RUW> struct WideWave {   // RUW: 16-row units of a block, 8 or 4
    static constexpr int NP = KFrag<D>::NP;
    static constexpr int R = RUW * 16;
    static constexpr int GROUPS = RUW / kWaveRows;      // groups of 32 window rows
    static constexpr int PARTS = kWaves / GROUPS;       // parts of a round's keys; a wave meets one part with one group
    static constexpr int TILES = kWaves / PARTS;        // 16-key tiles of a part
    static_assert(TILES == 4 || TILES == 2, "the exchange of the votes is written for these");
    const WideArgs<N>& A;
    const int tid, lane, n16, kg, w, rg, kp;
    // paged K: the page id the next request uses, asked for one round ahead of it
    int32_t page_id = 0;
    int in_page = 0;

    __device__ __forceinline__ WideWave(const WideArgs<N>& a)
        : A(a), tid(threadIdx.x), lane(threadIdx.x & 63), n16(threadIdx.x & 15), kg((threadIdx.x & 63) >> 4),
          w(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)), rg(w % GROUPS), kp(w / GROUPS) {}

    __device__ __forceinline__ int64_t round_key(const Cursor& c) const { return ((int64_t)c.sl * c.RPS + c.rd) * kRound; }
    __device__ __forceinline__ int64_t paged_row(int64_t pg, int in) const {   // ids outside the table: see physical_row
        pg = pg < 0 ? 0 : (pg >= A.pages ? A.pages - 1 : pg);
        return pg * A.page + in;
    }
    __device__ __forceinline__ int64_t row_of(const Cursor& c, int64_t j) const {   // keys past the end: the last row
        j = j < c.L ? j : c.L - 1;
        if constexpr (PAGED) {
            const unsigned l = (unsigned)(j + A.row0);
            return paged_row(A.table[l / (unsigned)A.page], (int)(l % (unsigned)A.page));
        }
        return j;
    }
    __device__ __forceinline__ void load_row(KFrag<D>& f, const Cursor& c, int64_t row) const {
        const char* p = c.kb + row * A.k_rs + kg * 16;
#pragma unroll
        for (int x = 0; x < NP; ++x) f.v[x] = *reinterpret_cast<const uint4*>(p + 64 * x);
    }
    __device__ __forceinline__ void ask_page(const Cursor& c) {
        if constexpr (PAGED) {
            unsigned j = (unsigned)round_key(c) + w * 16 + n16;      // (logical rows are below 2^31)
            j = (j < (unsigned)c.L ? j : (unsigned)c.L - 1) + (unsigned)A.row0;
            page_id = A.table[j / (unsigned)A.page];
            in_page = (int)(j % (unsigned)A.page);
        }
    }
    // This wave's tile of the cursor's round, and the cursor moved on.  Unconditional (see row_of).
    __device__ __forceinline__ KFrag<D> request(Cursor& c) {
        const Cursor at = c;
        advance(A, c);
        return request(at, c);
    }
    __device__ __forceinline__ KFrag<D> request(const Cursor& at, const Cursor& c) {   // c: the request after this one
        KFrag<D> f;
        int64_t row;
        if constexpr (PAGED) {
            row = paged_row(page_id, in_page);
            ask_page(c);
        } else {
            row = row_of(at, round_key(at) + w * 16 + n16);
        }
        load_row(f, at, row);
        __builtin_amdgcn_sched_barrier(0);
        return f;
    }
    // The wave's Q rows (MFMA fragments).  Padding rows repeat a valid one and are ignored later.
    __device__ __forceinline__ void load_q(KFrag<D> (&q)[kWaveRows], const Cursor& c) const {
        const WideEntry& E = A.e[c.e];
        int at = n16;
        asm volatile("" : "+v"(at));     // (rows addressed afresh for every unit: kept over the rounds they cost registers)
#pragma unroll
        for (int i = 0; i < kWaveRows; ++i) {
            const int ru = rg * kWaveRows + i;
            const int rh = ru * A.inv_uh >> 8;
            int head = c.blk * A.hb + rh, row = (ru - rh * A.UH) * 16 + at;
            head = head < A.g ? head : A.g - 1;
            row = row < A.W ? row : A.W - 1;
            const char* p = E.q + (((int64_t)c.kv * A.g + head) * A.W + row) * (D * 2) + kg * 16;
#pragma unroll
            for (int x = 0; x < NP; ++x) q[i].v[x] = *reinterpret_cast<const uint4*>(p + 64 * x);
        }
    }
    // Prompt-phase causal mask of the 16 keys from j0 on (keys x rows) against row unit i of the wave: row x does not see keys
    // after n + x (which for a real row covers the keys past the end; what padding rows hold is ignored).
    __device__ __forceinline__ void mask(wf32x4& a, int j0, int i, const Cursor& c) const {
        const int ru = rg * kWaveRows + i, d = j0 - c.n + kg * 4 - n16 - (ru - (ru * A.inv_uh >> 8) * A.UH) * 16;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (d + r > 0) a[r] = -INFINITY;
    }
    __device__ __forceinline__ void keep(uint4* buf, const KFrag<D>& f) const {   // the wave's tile into the round's buffer
#pragma unroll
        for (int x = 0; x < NP; ++x) buf[(w * NP + x) * 64 + lane] = f.v[x];
    }
    __device__ __forceinline__ void tile(KFrag<D>& f, const uint4* buf, int t) const {   // tile t of the wave's part
#pragma unroll
        for (int x = 0; x < NP; ++x) f.v[x] = buf[((kp * TILES + t) * NP + x) * 64 + lane];
    }
};

// The sums of exponentials of a lane's two rows (n16 of the wave's two row units) relative to their references.  Logits are taken keys x
// rows: a lane has four keys (4 * kg + r) of one row, so that the sums over keys need no exchange between lanes but for the four of a
// row, once a slice.
template <typename T, int D, int RUW, typename Wv> struct RowSums {
    static_assert(kWaveRows == 2, "the rows of a lane are written out");
    static constexpr int kFirst = RUW == 8 ? 4 : 16;    // keys that the references come from
    const Wv& W;
    const KFrag<D> (&q)[kWaveRows];
    float z[kWaveRows], ref[kWaveRows], neg[kWaveRows];  // neg: minus the rows' origins (RUW = 4)
    bool raised = false;                                // (wave-uniform) a reference was raised since it was last put back

    __device__ __forceinline__ RowSums(const Wv& w, const KFrag<D> (&q_)[kWaveRows]) : W(w), q(q_) {}
    __device__ __forceinline__ wf32x4 start(int i) const {
        const float v = kOrigin<RUW> ? neg[i] : 0.f;
        return wf32x4{v, v, v, v};
    }
    // The rows' origins and references from the prompt's first kFirst keys (or fewer: those that every row sees; each row of lanes
    // brings all of them).  They depend on the unit alone.
    __device__ __forceinline__ void ask_first(KFrag<D>& f, const Cursor& c) const {
        const int j = W.n16 & (kFirst - 1);
        W.load_row(f, c, W.row_of(c, j < c.n ? j : c.n));
    }
    __device__ __forceinline__ void begin(const KFrag<D>& f) {
#pragma unroll
        for (int i = 0; i < kWaveRows; ++i) {
            const wf32x4 a = logits16<T, D>(f, q[i]);
            float m = fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3]));   // (four keys: every lane of the row has them)
            if constexpr (kOrigin<RUW>) {   // of the four quads' maxima the second largest is the origin
                const Two x = swap32(m, m);
                const float hi = fmaxf(x.a, x.b), lo = fminf(x.a, x.b);
                const Two h = swap16(hi, hi), l = swap16(lo, lo);
                float o = fmaxf(fminf(h.a, h.b), fmaxf(l.a, l.b));
                o = fabsf(o) < 0x1p100f ? o : 0.f;
                neg[i] = -o;
                m = fmaxf(h.a, h.b) - o;
            }
            m *= W.A.c2;
            ref[i] = m == -INFINITY ? 0.f : m;
            z[i] = 0.f;
        }
    }
    // A round's keys (in buf), which begin with the cursor's.
    __device__ __forceinline__ void round(const uint4* buf, const Cursor& cc) {
        constexpr int TILES = Wv::TILES;
        const float c2 = W.A.c2;
        const int j0 = (int)W.round_key(cc) + W.kp * (TILES * 16);   // (prompts have less than 2^31 keys)
        const bool special = j0 + TILES * 16 > cc.n;   // window columns or keys past the end among the wave's
        float y[kWaveRows];              // the round's sums
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            KFrag<D> f;
            W.tile(f, buf, t);
#pragma unroll
            for (int i = 0; i < kWaveRows; ++i) {
                wf32x4 a = logits16<T, D>(f, q[i], start(i));
                if (special) W.mask(a, j0 + t * 16, i, cc);
                float x[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) x[r] = __builtin_amdgcn_exp2f(fmaf(a[r], c2, -ref[i]));
                const float sum = (x[0] + x[1]) + (x[2] + x[3]);
                y[i] = t == 0 ? sum : y[i] + sum;
            }
            __builtin_amdgcn_sched_barrier(0);   // (one tile at a time: more do not fit the registers)
        }
        if (__any(fmaxf(y[0], y[1]) > kRaiseAt)) {   // some row's logits lie far above its reference: first their maxima, then the sums again
            raised = true;
            auto each = [&](auto f2) __attribute__((always_inline)) {
#pragma clang loop unroll(disable)
                for (int t = 0; t < TILES; ++t) {
                    KFrag<D> f;
                    W.tile(f, buf, t);
#pragma unroll
                    for (int i = 0; i < kWaveRows; ++i) {
                        wf32x4 a = logits16<T, D>(f, q[i], start(i));
                        W.mask(a, j0 + t * 16, i, cc);
                        f2(a, i);
                    }
                }
            };
            y[0] = y[1] = -INFINITY;
            each([&](const wf32x4& a, int i) __attribute__((always_inline)) { y[i] = fmaxf(fmaxf(y[i], fmaxf(a[0], a[1])), fmaxf(a[2], a[3])); });
#pragma unroll
            for (int i = 0; i < kWaveRows; ++i) {
                const float m = rows_max(y[i]) * c2, to = m > ref[i] + kRaiseMin ? m - kRaiseBelow : ref[i];
                z[i] *= __builtin_amdgcn_exp2f(ref[i] - to);
                ref[i] = to;
                y[i] = 0.f;
            }
            each([&](const wf32x4& a, int i) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < 4; ++r) y[i] += __builtin_amdgcn_exp2f(fmaf(a[r], c2, -ref[i]));
            });
        }
        z[0] += y[0];
        z[1] += y[1];
    }
    // The sums over the four lanes of a row, and the references: st[0] and st[1], a part's rows one behind the other.
    __device__ __forceinline__ void leave(float* ref_to, float* sum_to, float* origin_to) const {
        const float sum = halves(z[0], z[1]);   // lanes 0-31: the first row's, of two of its four lanes; 32-63 the second's
        const float all = quarters(sum, sum);
        if ((W.kg & 1) == 0) {           // (a lane for each row)
            const int second = W.kg >> 1, at = (W.rg * kWaveRows + second) * 16 + W.n16;
            ref_to[at] = second ? ref[1] : ref[0];
            sum_to[at] = all;
            if constexpr (kOrigin<RUW>)
                if (origin_to) origin_to[at] = second ? neg[1] : neg[0];
        }
    }
};

// The parts' sums of a row added up in a fixed order: (reference, sum).
template <int PARTS, int R> __device__ __forceinline__ float2 add_parts(const float (&ref)[PARTS][R], const float (&sum)[PARTS][R], int row) {
    float m = -INFINITY, s = 0.f;
#pragma unroll
    for (int v = 0; v < PARTS; ++v) m = fmaxf(m, ref[v][row]);
#pragma unroll
    for (int v = 0; v < PARTS; ++v) s += sum[v][row] * __builtin_amdgcn_exp2f(ref[v][row] - m);
    return make_float2(m, s);
}

// (reference, sum) pairs merged in a balanced tree (fixed order, few roundings)
template <int n> __device__ __forceinline__ void fold(const float2 (&y)[n], float& m, float& s) {
    float t[n];
    m = -INFINITY;
#pragma unroll
    for (int i = 0; i < n; ++i) m = fmaxf(m, y[i].y != 0.f ? y[i].x : -INFINITY);
#pragma unroll
    for (int i = 0; i < n; ++i) t[i] = y[i].y != 0.f ? y[i].y * __builtin_amdgcn_exp2f(y[i].x - m) : 0.f;
#pragma unroll
    for (int d = 1; d < n; d <<= 1)
#pragma unroll
        for (int i = 0; i + d < n; i += 2 * d) t[i] += t[i + d];
    s = t[0];
}

// Sums over the rows of a row unit of the votes on a round's keys (in buf), into sm_v; logits are taken rows x keys.
// mref and wgt: the rows' reference and 1 / sum (padding rows: +inf and 0).
template <typename T, int D, int RUW, typename Wv>
__device__ __forceinline__ void round_votes(const Wv& W, const KFrag<D> (&q)[kWaveRows], const Origins<RUW>& org, const float (&mref)[kWaveRows][4],
                                            const float (&wgt)[kWaveRows][4], const uint4* buf, float (&sm_v)[RUW][kRound]) {
    constexpr int TILES = Wv::TILES;
    const float c2 = W.A.c2;
    float v[kWaveRows][TILES];
#pragma unroll
    for (int t = 0; t < TILES; ++t) {
        KFrag<D> f;
        W.tile(f, buf, t);
#pragma unroll
        for (int i = 0; i < kWaveRows; ++i) {
            const wf32x4 a = org.template logits<T, D>(q[i], f, i);
            float s = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) s = fmaf(__builtin_amdgcn_exp2f(fmaf(a[r], c2, -mref[i][r])), wgt[i][r], s);
            v[i][t] = s;
        }
        if (t & 1) __builtin_amdgcn_sched_barrier(0);
    }
    // sums over the four lanes of a column: pairs of tiles share the exchanges, so that a lane ends with one tile's
    if constexpr (TILES == 4) {
#pragma unroll
        for (int i = 0; i < kWaveRows; ++i)
            sm_v[W.rg * kWaveRows + i][W.kp * (TILES * 16) + ((W.kg >> 1) + 2 * (W.kg & 1)) * 16 + W.n16] =
                quarters(halves(v[i][0], v[i][1]), halves(v[i][2], v[i][3]));
    } else {                             // the wave's two row units share them too
        sm_v[W.rg * kWaveRows + (W.kg & 1)][W.kp * (TILES * 16) + (W.kg >> 1) * 16 + W.n16] =
            quarters(halves(v[0][0], v[0][1]), halves(v[1][0], v[1][1]));
    }
}
// A row's (reference, 1 / sum) from what its slices' merge came to.
template <int N> __device__ __forceinline__ float2 row_weight(const WideArgs<N>& A, const Cursor& cc, int row, float m, float s) {
    const int ru = row >> 4, rh = ru * A.inv_uh >> 8;
    const bool real = rh < A.hb && cc.blk * A.hb + rh < A.g && (ru - rh * A.UH) * 16 + (row & 15) < A.W && s > 0.f;
    return real ? make_float2(m, 1.0f / s) : make_float2(INFINITY, 0.f);
}
// Where a round's votes go: from the round's first key in the block's first query head's vote row on.
struct VoteRows {
    float* at = nullptr;
    int64_t pitch = 0;
    int keys = 0, heads = 0;
    template <typename Wv> __device__ __forceinline__ void aim(const Wv& W, const Cursor& cc) {
        const WideEntry& E = W.A.e[cc.e];
        const int h0 = cc.blk * W.A.hb;
        const int64_t k0 = W.round_key(cc);
        at = E.vote + ((int64_t)cc.kv * W.A.g + h0) * E.vpitch + k0;
        pitch = E.vpitch;
        keys = (int)(cc.n - k0 < kRound ? cc.n - k0 : kRound);
        heads = W.A.g - h0 < W.A.hb ? W.A.g - h0 : W.A.hb;
    }
    // The row units of every query head added up and stored.
    template <int RUW> __device__ __forceinline__ void store(const float (&sm_v)[RUW][kRound], int tid, int UH) const {
        const int key = tid % kRound;
        if (key < keys)
            for (int h = tid / kRound; h < heads; h += kThreads / kRound) {
                float s = sm_v[h * UH][key];
                for (int u = 1; u < UH; ++u) s += sm_v[h * UH + u][key];
                // (device scope: see the vote stores of the single-read kernel)
                __hip_atomic_store(at + (int64_t)h * pitch + key, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
    }
};

template <typename T, int D, bool PAGED, int N, int RUW>
__global__ __launch_bounds__(kThreads, 4) void wide_stats(const WideArgs<N> A) {
    using Wv = WideWave<T, D, PAGED, N, RUW>;
    constexpr int R = Wv::R, PARTS = Wv::PARTS;
    __shared__ uint4 kbuf[2][kWaves * Wv::NP * 64];                      // K of two rounds as MFMA fragments
    __shared__ float sm_base[PARTS][R];                                  // the references at a slice's start
    __shared__ float sm_ref[2][PARTS][R], sm_sum[2][PARTS][R], sm_org[2][kExtra<RUW> ? R : 1];   // two slices' references, sums and origins
    Wv W(A);
    {
        const int64_t wg = ((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x, all = (int64_t)gridDim.x * gridDim.y * gridDim.z * kThreads;
        for (int64_t i = wg * kThreads + W.tid; i < A.nzeros; i += all) A.zeros[i] = 0u;
        if (A.flag && wg == 0 && W.tid == 0) *A.flag = 0u;
    }
    int rounds;
    Cursor cc = begin_share<true>(A, rounds), pc = cc;
    if (rounds <= 0) return;
    KFrag<D> q[kWaveRows], S;
    RowSums<T, D, RUW, Wv> rs(W, q);

    // A unit begins; every slice starts from the unit's references, so its result does not depend on which slices its workgroup had before.
    float* const base = &sm_base[W.kp][W.rg * kWaveRows * 16 + W.n16];   // the lane's first row (its four lanes hold the same)
    auto ask_unit = [&](KFrag<D>& f) __attribute__((always_inline)) {
        W.load_q(q, cc);
        rs.ask_first(f, cc);
    };
    auto begin_unit = [&](const KFrag<D>& f) __attribute__((always_inline)) {
        rs.begin(f);
        base[0] = rs.ref[0];
        base[16] = rs.ref[1];
    };
    int par = 0;                         // which half of sm_ref and sm_sum the current slice uses
    float2* pending = nullptr;           // where the pairs of the slice before go, once all waves have left theirs,
    float2* origins = nullptr;           //   and the unit's origins (with its first slice)
    auto store_slice = [&](int half) __attribute__((always_inline)) {
        if (W.tid < R) {
            pending[W.tid] = add_parts<PARTS, R>(sm_ref[half], sm_sum[half], W.tid);
            if constexpr (kOrigin<RUW>)
                if (origins) origins[W.tid] = make_float2(sm_org[half][W.tid], 0.f);
        }
        pending = nullptr;
    };

    KFrag<D> first;
    W.ask_page(pc);
    ask_unit(first);
    S = W.request(pc);
    begin_unit(first);
    int left = rounds;
    // A round: its keys go from the landing registers to LDS, the next round is requested, and every wave meets its
    // part of the keys with its rows.
    for (int half = 0;; half ^= 1) {
        W.keep(kbuf[half], S);
        S = W.request(pc);
        lds_meet();
        if (pending) store_slice(par ^ 1);
        rs.round(kbuf[half], cc);
        --left;
        if (cc.rd + 1 == cc.RPS) {       // the slice's last round
            rs.leave(sm_ref[par][W.kp], sm_sum[par][W.kp], W.kp == 0 ? sm_org[par] : nullptr);
            if (rs.raised) {
                rs.ref[0] = base[0];
                rs.ref[1] = base[16];
            }
            rs.raised = false;
            rs.z[0] = rs.z[1] = 0.f;
            pending = A.e[cc.e].part + unit_part<RUW>(A, cc) + (int64_t)cc.sl * R;
            if constexpr (kOrigin<RUW>) origins = cc.sl == 0 ? pending + (int64_t)cc.NS * R : nullptr;
            par ^= 1;
        }
        if (left <= 0) break;
        if (advance(A, cc)) {
            ask_unit(first);
            begin_unit(first);
        }
    }
    lds_meet();
    store_slice(par ^ 1);                // (a workgroup's share ends with a slice)
}

template <typename T, int D, bool PAGED, int N, int RUW>
__global__ __launch_bounds__(kThreads, 4) void wide_votes(const WideArgs<N> A) {
    using Wv = WideWave<T, D, PAGED, N, RUW>;
    constexpr int R = Wv::R, SUB = kThreads / R;   // SUB threads share a row in the merge of its slices
    __shared__ uint4 kbuf[2][kWaves * Wv::NP * 64];
    __shared__ float sm_v[2][RUW][kRound];                            // sums over the rows of a row unit, per key
    __shared__ float2 sm[SUB][R];
    __shared__ __attribute__((aligned(16))) float2 smf[R];
    __shared__ __attribute__((aligned(16))) float smo[kOrigin<RUW> ? R : 1];
    Wv W(A);
    int rounds;
    Cursor cc = begin_share<false>(A, rounds), pc = cc;
    if (rounds <= 0) return;
    KFrag<D> q[kWaveRows], S;
    W.ask_page(pc);
    S = W.request(pc);

    Origins<RUW> org;
    float mref[kWaveRows][4], wgt[kWaveRows][4];   // the rows' reference and 1 / sum (padding rows: +inf and 0)
    auto begin_unit = [&]() __attribute__((always_inline)) {            // the unit's slices merged in a fixed order, and the wave's Q rows
        const int row = W.tid % R, sub = W.tid / R;
        const float2* src = A.e[cc.e].part + unit_part<RUW>(A, cc) + row;
        float m = -INFINITY, s = 0.f;
#pragma clang loop unroll(disable)
        for (int s0 = sub; s0 < cc.NS; s0 += 8 * SUB) {   // eight slices' pairs in flight at a time
            float2 x[9];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int sl = s0 + i * SUB;
                x[i] = sl < cc.NS ? src[(int64_t)sl * R] : make_float2(-INFINITY, 0.f);
            }
            x[8] = make_float2(m, s);
            fold(x, m, s);
        }
        sm[sub][row] = make_float2(m, s);
        if constexpr (kOrigin<RUW>)
            if (W.tid < R) smo[row] = src[(int64_t)cc.NS * R].x;
        W.load_q(q, cc);
        lds_meet();
        if (W.tid < R) {
            float2 y[SUB];
#pragma unroll
            for (int i = 0; i < SUB; ++i) y[i] = sm[i][W.tid];
            fold(y, m, s);
            smf[W.tid] = row_weight(A, cc, W.tid, m, s);
        }
        lds_meet();
#pragma unroll
        for (int i = 0; i < kWaveRows; ++i) {
            const float4* f4 = reinterpret_cast<const float4*>(&smf[(W.rg * kWaveRows + i) * 16 + W.kg * 4]);
            const float4 a = f4[0], b = f4[1];
            mref[i][0] = a.x, wgt[i][0] = a.y, mref[i][1] = a.z, wgt[i][1] = a.w;
            mref[i][2] = b.x, wgt[i][2] = b.y, mref[i][3] = b.z, wgt[i][3] = b.w;
            if constexpr (kOrigin<RUW>) org.neg[i] = *reinterpret_cast<const wf32x4*>(&smo[(W.rg * kWaveRows + i) * 16 + W.kg * 4]);
        }
    };
    begin_unit();

    VoteRows last;                       // of the round before
    int left = rounds;
    for (int half = 0;; half ^= 1) {
        W.keep(kbuf[half], S);
        S = W.request(pc);
        lds_meet();
        last.template store<RUW>(sm_v[half ^ 1], W.tid, A.UH);
        round_votes<T, D, RUW>(W, q, org, mref, wgt, kbuf[half], sm_v[half]);
        last.aim(W, cc);
        --left;
        if (left <= 0) break;
        if (advance(A, cc)) begin_unit();
    }
    lds_meet();
    last.template store<RUW>(sm_v[(rounds & 1) ^ 1], W.tid, A.UH);
}

// Both passes in one launch, where a call's slices all find a place at once (one prompt, a workgroup per slice): a slice's keys
// are met twice by its own workgroup, which hands its rows' (reference, sum) to the unit's others in between as
// words that validate themselves (see snapkv_handoff.h).  The two last rounds' keys are still in LDS then, Q in registers, and the round
// before those on its way.  The arithmetic and its order are those of the two launches, and so are the votes, bit for bit.
// A pass of a short call is bound by its start and its end (20 us at 28471 keys, 32/8 heads, of which about 11 are arithmetic and 10 the
// stream, side by side): the second one's start, its Q and the keys of two of its three or four rounds are saved, for one exchange between workgroups.
// Microseconds per call, two launches / one (8 KV heads of four query heads, W = 32): 18500 keys 51.3 / 44.6; 24000 52.9 / 45.7; 32768 57.2 / 51.2;
// 65536 80.2 / 71.2; 131072 128.7 / 114.0; one KV head 18500 35.0 / 32.0, 131072 48.1 / 45.0; on a caller's workspace, whose words a
// launch before this one has to make ready (the first of two passes cleared the selection's counters on the way), 28471 keys 56.0 / 51.3.
// Of keys that no cache holds (a rotation over 2 GB of prompts), before the prompt came here or in two launches / one: 17300 keys 59.5 / 45.9; 28471 59.2 / 52.3;
// 65536 92.9 / 84.8; W = 64: 12300 59.2 / 47.7; 131072 219 / 199; one KV head 18433 34.2 / 31.4.  Counters (profiles/sq_counters_gqa_two_pass.txt), 32768 keys:
// of 79 thousand cycles a SIMD's matrix unit is busy for 17 and its vector instructions take 34; 101 MB are read for 67 of keys.
// Blocks of 64 rows, which begin at 131073 keys, keep the two launches, and so do the prompts of a batch that has two or more of this kind.
//
// No workgroup depends on another's being resident: other streams' kernels may hold its place, or wait for ours.  One that has polled for
// kPatience takes the statistics of a missing slice itself, with the same instructions and so the same words (whose
// writer is of no consequence), looks again without waiting, and in the end takes its own slice once more, so that the votes find LDS as they
// expect it.  Workgroups take different slices (see snapkv_help.h), so that a unit of which r workgroups have places and m have none is
// done after kPatience and 2 m / r + 2 slices' statistics at most or so, even if the others' places are not free until then: half a millisecond
// and, in the worst case of one workgroup with a place, the statistics of the whole unit, where two launches would have gone on with what places there are.
constexpr unsigned kPatience = 1u << 9;      // polls (about half a millisecond)
template <typename T, int D, bool PAGED>
__global__ __launch_bounds__(kThreads, 4) void wide_once(const WideArgs<1> A) {
    constexpr int RUW = 8;
    using Wv = WideWave<T, D, PAGED, 1, RUW>;
    constexpr int R = Wv::R, PARTS = Wv::PARTS, SUB = kThreads / R;
    __shared__ uint4 kbuf[2][kWaves * Wv::NP * 64];
    struct Sums {
        float ref[PARTS][R], sum[PARTS][R];
    };
    union Left {                         // (the slice's sums have been read when the first votes are left)
        Sums sums;
        float votes[2][RUW][kRound];
    };
    __shared__ Left sm;
    __shared__ float2 sm_part[SUB][R];
    __shared__ __attribute__((aligned(16))) float2 smf[R];
    __shared__ int sm_missing;           // of the slices whose words somebody missed the smallest key
    Wv W(A);
    int rounds;
    Cursor cc = begin_share<true>(A, rounds);
    const int own = cc.sl;
    KFrag<D> q[kWaveRows], S;
    // Requests: the rounds from the first to the last, then back from the one before the last two to the first.
    Cursor pc = cc;
    int asked = 0;
    auto request = [&]() __attribute__((always_inline)) {
        const Cursor at = pc;
        ++asked;
        const int back = 2 * rounds - 3 - asked;
        pc.rd = asked < rounds ? asked : (back > 0 ? back : 0);
        return W.request(at, pc);
    };
    W.load_q(q, cc);
    float2* const words = A.e[0].part + ((int64_t)cc.kv * A.nblk + cc.blk) * cc.NS * R;
    bool gave_up = false;
    for (int turn = 0;; ++turn) {        // (once, but for workgroups that lost their patience)
        int none = 0;                    // (what is computed from it is computed in the loop: no register holds it meanwhile)
        asm volatile("" : "+s"(none));
        const int tid = W.tid + none;
        RowSums<T, D, RUW, Wv> rs(W, q);
        KFrag<D> first;
        pc = cc;
        pc.rd = asked = 0;
        W.ask_page(pc);
        rs.ask_first(first, cc);
        S = request();
        rs.begin(first);
        for (int r = 0; r < rounds; ++r) {
            W.keep(kbuf[r & 1], S);
            S = request();
            lds_meet();
            cc.rd = r;
            rs.round(kbuf[r & 1], cc);
        }
        rs.leave(sm.sums.ref[W.kp] + none, sm.sums.sum[W.kp] + none, nullptr);
        if (tid == 0) sm_missing = kNoneMissing;
        lds_meet();
        if (tid < R) {
            const float2 x = add_parts<PARTS, R>(sm.sums.ref, sm.sums.sum, tid);
            publish_pair(words + (int64_t)cc.sl * R + tid, x.x, x.y);
        }
        if (turn) {                      // (these words are the next ones to be looked for)
            __threadfence();
            lds_meet();
        }
        // The unit's slices merged in the order of wide_votes.
        const int row = tid % R, sub = tid / R;
        const float2* const src = words + row;
        const unsigned limit = patience(turn, A.spin_limit);
        float m = -INFINITY, s = 0.f;
        bool missed = false;
#pragma clang loop unroll(disable)
        for (int s0 = sub; s0 < cc.NS; s0 += 8 * SUB) {
            unsigned long long bits[8];
            float2 x[9];
#pragma unroll
            for (int i = 0; i < 8; ++i) bits[i] = load_pair_bits(src + (int64_t)(s0 + i * SUB < cc.NS ? s0 + i * SUB : 0) * R);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                float pm = -INFINITY, ps = 0.f;
                if (s0 + i * SUB < cc.NS) {
                    unpack_pair(await_pair(src + (int64_t)(s0 + i * SUB) * R, bits[i], limit, missed), pm, ps);
                    if (missed && bits[i] == kInvalidPair) atomicMin(&sm_missing, help_key(s0 + i * SUB, own));
                }
                x[i] = make_float2(pm, ps);
            }
            x[8] = make_float2(m, s);
            fold(x, m, s);
        }
        sm_part[sub][row] = make_float2(m, s);
        lds_meet();
        const int key = __builtin_amdgcn_readfirstlane(sm_missing);
        const bool none_missing = key == kNoneMissing;
        gave_up = !none_missing && turn > 2 * cc.NS;     // (a bound only: every turn leaves the words of one slice, so it is not reached)
        const int next = none_missing || gave_up ? own : help_slice(key, own);
        if (tid < R) {
            float2 y[SUB];
#pragma unroll
            for (int i = 0; i < SUB; ++i) y[i] = sm_part[i][tid];
            fold(y, m, s);
            smf[tid] = row_weight(A, cc, tid, m, s);
        }
        lds_meet();
        if (next == cc.sl && (none_missing || gave_up)) break;
        cc.sl = next;
    }
    Origins<RUW> org;
    float mref[kWaveRows][4], wgt[kWaveRows][4];
#pragma unroll
    for (int i = 0; i < kWaveRows; ++i) {
        const float4* f4 = reinterpret_cast<const float4*>(&smf[(W.rg * kWaveRows + i) * 16 + W.kg * 4]);
        const float4 a = f4[0], b = f4[1];
        mref[i][0] = a.x, wgt[i][0] = a.y, mref[i][1] = a.z, wgt[i][1] = a.w;
        mref[i][2] = b.x, wgt[i][2] = b.y, mref[i][3] = b.z, wgt[i][3] = b.w;
    }
    VoteRows last;
    for (int i = 0; i < rounds; ++i) {
        const int r = rounds - 1 - i;
        if (i >= 2) {                    // (the last two are in LDS; everybody has left the buffer of the round two before)
            W.keep(kbuf[r & 1], S);
            S = request();
        }
        lds_meet();
        last.template store<RUW>(sm.votes[(i & 1) ^ 1], W.tid, A.UH);
        cc.rd = r;
        round_votes<T, D, RUW>(W, q, org, mref, wgt, kbuf[r & 1], sm.votes[i & 1]);
        last.aim(W, cc);
    }
    lds_meet();
    last.template store<RUW>(sm.votes[(rounds & 1) ^ 1], W.tid, A.UH);
    if (gave_up) {
        atomicAdd(&g_wide_timeouts, 1u);
        if (A.gave_up) __hip_atomic_store(A.gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

struct Blocks {
    int ru, UH, hb, nblk;                // 16-row units of a block (8 or 4) and of a query head, query heads of a block, blocks
};
bool row_blocks(const ScoreGeom& G, Blocks* b) {
    b->UH = (G.W + 15) / 16;
    const int units = G.g * b->UH;
    if (b->UH > 8 || (units < 8 && units != 4)) return false;   // (64 window rows per KV head, or at least 128)
    b->ru = units == 4 ? 4 : 8;
    const int most = std::min(G.g, b->ru / b->UH);
    b->nblk = (G.g + most - 1) / most;
    b->hb = (G.g + b->nblk - 1) / b->nblk;   // blocks of about equal size
    return true;
}

// Rounds per slice and slices per unit.  They depend on the prompt and its own heads only, not on what else the call holds.
// A prompt of more than kPlacesAll / kSlices units of 128 rows has as many slices per unit as still find a place all at once, so that it takes one
// launch (wide_once).  Microseconds per call, 64 slices / this: 8 KV heads, W = 64, four query heads (16 units): 6200 keys 50.2 / 38.9;
// 12300: 56.0 / 46.9;  28000: 77.7 / 60.6;  131072: 192.8 / 179.8;  12 units of W = 32: 20000: 62.1 / 48.9;  131072: 210 / 185;  32 units of
// W = 128: 20000: 95 / 77;  131072: 453 / 428.  Layers of one call walk the same slices (a head's result is the same in every call), of which
// each workgroup then has few and long ones; with the votes shared out by rounds and the statistics' shares as share_of says (snapkv_shares.h) that
// is mostly the same or faster.  16 units, 2 layers: 8500 keys 64 / 67;  12300: 72.9 / 74.7;  20000: 91 / 83;  32000: 122 / 112;  3: 8500: 81 / 79;  12300: 94 / 93;
// 17000: 113 / 113;  20000: 123 / 122;  4: 10500: 101 / 99;  15000: 122 / 114;  24000: 166 / 153;  32000: 209 / 199;  6: 10500: 134 / 133;  17000: 182 / 181;  32000: 347 / 339;
// 12 units: 2: 16384: 83 / 79;  3: 28000: 136 / 140.  A lane's sums run over up to four times as many rounds (32 units): the votes' error against float64, over
// 24 settings, was 1.002 of that with 64 slices on average and at most 1.037, which is what the settings scatter by.
int rounds_per_slice(const ScoreGeom& G, const Blocks& b) {
    auto rounds = [&](int64_t most) { return (G.L + kRound * most - 1) / (kRound * most); };
    const int64_t units = (int64_t)G.own_kv * b.nblk;
    const int64_t most = b.ru == 8 && units * kSlices > kPlacesAll && units <= kMaxOnce ? kPlacesAll / units : kSlices;
    const int64_t usual = rounds(most), few_units = rounds(std::max(most, kPlaces / units));
    return (int)std::max(few_units, std::min<int64_t>(usual, 2));   // (a slice's end costs half a round)
}
int slices_of(const ScoreGeom& G, const Blocks& b) {
    const int64_t keys = (int64_t)rounds_per_slice(G, b) * kRound;
    return (int)((G.L + keys - 1) / keys);
}

int wide_cus() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
        cached[dev] = n;
    }
    return cached[dev];
}

template <int N> WideArgs<N> first_entries(const WideArgs<kMaxWide>& all) {
    WideArgs<N> A;
    A.count = all.count, A.direct = all.direct, A.g = all.g, A.W = all.W, A.UH = all.UH, A.hb = all.hb, A.nblk = all.nblk, A.inv_uh = all.inv_uh;
    A.c2 = all.c2, A.k_rs = all.k_rs, A.table = all.table, A.page = all.page, A.pages = all.pages, A.row0 = all.row0;
    A.rounds = all.rounds, A.share = all.share, A.more = all.more, A.reversed = all.reversed, A.zeros = all.zeros, A.nzeros = all.nzeros, A.flag = all.flag;
    A.spin_limit = all.spin_limit, A.gave_up = all.gave_up;
    for (int i = 0; i < N; ++i) A.e[i] = all.e[i];
    return A;
}

template <typename T, int D>
hipError_t launch_once(const WideArgs<kMaxWide>& all, bool paged, dim3 grid, hipStream_t st) {
    const WideArgs<1> A = first_entries<1>(all);
    if (paged) hipLaunchKernelGGL((wide_once<T, D, true>), grid, dim3(kThreads), 0, st, A);
    else hipLaunchKernelGGL((wide_once<T, D, false>), grid, dim3(kThreads), 0, st, A);
    stage_done(st, kStageWide);
    return hipGetLastError();
}

template <typename T, int D, bool PAGED, int N, int RUW>
hipError_t launch_both(const WideArgs<kMaxWide>& all, dim3 grid, hipStream_t st) {
    const WideArgs<N> A = first_entries<N>(all);
    hipLaunchKernelGGL((wide_stats<T, D, PAGED, N, RUW>), grid, dim3(kThreads), 0, st, A);
    hipLaunchKernelGGL((wide_votes<T, D, PAGED, N, RUW>), grid, dim3(kThreads), 0, st, A);
    stage_done(st, kStageWide);    // (both launches)
    return hipGetLastError();
}
template <typename T, int D, int RUW> hipError_t by_entries(const WideArgs<kMaxWide>& A, dim3 grid, hipStream_t st) {
    if (A.count > 1) return launch_both<T, D, false, kMaxWide, RUW>(A, grid, st);
    return A.table ? launch_both<T, D, true, 1, RUW>(A, grid, st) : launch_both<T, D, false, 1, RUW>(A, grid, st);
}
template <typename T, int D> hipError_t by_rows(const WideArgs<kMaxWide>& A, int ru, dim3 grid, hipStream_t st) {
    return ru == 4 ? by_entries<T, D, 4>(A, grid, st) : by_entries<T, D, 8>(A, grid, st);
}

}  // namespace

// Whether these kernels take the prompt: enough window rows and keys (min_row_keys), and statistics that fit what a workspace
// holds anyway (a region of the streaming passes, or the pooled scores that come later).  The answer depends on the prompt and on the KV heads of a
// layer (own_kv), not on how many layers or prompts a call has: the place is looked at for one head.
static bool wide_shape(const ScoreGeom& G, Blocks* b) {
    if (G.n <= 0 || !row_blocks(G, b)) return false;
    const int64_t least = b->ru == 8 ? min_row_keys((int64_t)G.own_kv * b->nblk) : b->UH == 2 ? kMinRowKeys64of2 : kMinRowKeys64;
    if ((int64_t)G.g * b->UH * 16 * G.L < least) return false;
    ScoreGeom one = G;
    one.Hkv = 1;
    const size_t part = sizeof(float2) * (size_t)b->nblk * (slices_of(G, *b) + (b->ru == 4 ? kExtra<4> : kExtra<8>)) * b->ru * 16;
    return part <= std::max(stream_stat_bytes(one), sizeof(float) * (size_t)G.g * (size_t)G.n);
}

bool wide_ok(int dtype, int D, const ScoreGeom& G) {
    Blocks b;
    if ((dtype != 0 && dtype != 2) || (D != 64 && D != 128) || !wide_shape(G, &b)) return false;
    return (int64_t)G.Hkv * b.nblk * slices_of(G, b) * rounds_per_slice(G, b) <= kMaxRounds;
}

size_t wide_part_bytes(const ScoreGeom& G) {
    Blocks b;
    if (!wide_shape(G, &b)) return 0;
    return (sizeof(float2) * (size_t)G.Hkv * b.nblk * (slices_of(G, b) + (b.ru == 4 ? kExtra<4> : kExtra<8>)) * b.ru * 16 + 255) & ~(size_t)255;
}

static hipError_t score_wide(int dtype, int D, int count, const WidePrompt* P, hipStream_t st, const WideClear& clear, bool once, unsigned* gave_up) {
    if (count < 1 || count > kMaxWide) return hipErrorInvalidValue;
    for (int i = 0; i < count; ++i)
        if (!P[i].q || !P[i].k || !P[i].vote || !P[i].part) return hipErrorInvalidValue;
    Blocks b;
    if ((dtype != 0 && dtype != 2) || (D != 64 && D != 128) || !row_blocks(*P[0].G, &b)) return hipErrorInvalidValue;
    const ScoreGeom& G0 = *P[0].G;
    if (G0.k_table && count != 1) return hipErrorInvalidValue;
    WideArgs<kMaxWide> A;
    A.count = count;
    A.g = G0.g;
    A.W = G0.W;
    A.UH = b.UH;
    A.hb = b.hb;
    A.nblk = b.nblk;
    A.inv_uh = (256 + b.UH - 1) / b.UH;
    A.c2 = G0.c2;
    A.k_rs = G0.k_rs;
    A.table = G0.k_table;
    A.page = G0.k_page;
    A.pages = G0.k_pages;
    A.row0 = G0.k_row0;
    A.rounds = 0;
    A.zeros = clear.zeros;
    A.nzeros = clear.zeros ? clear.nzeros : 0;
    A.flag = clear.flag;
    A.spin_limit = wait_limit(kPatience);
    A.gave_up = gave_up;
    int64_t slices = 0;
    bool alike = true;                   // all slices are of the same length, as those of layers are
    for (int i = 0; i < count; ++i) {
        const ScoreGeom& G = *P[i].G;
        if (G.g != G0.g || G.W != G0.W || G.k_rs != G0.k_rs || G.n <= 0 || G.L + G.k_row0 >= (int64_t)1 << 31) return hipErrorInvalidValue;
        WideEntry& E = A.e[i];
        E.q = static_cast<const char*>(P[i].q);
        E.k = static_cast<const char*>(P[i].k);
        E.vote = P[i].vote;
        E.part = P[i].part;
        E.k_hs = G.k_hs;
        E.vpitch = G.vpitch;
        E.round_begin = A.rounds;
        E.L = (int)G.L;
        E.n = (int)G.n;
        E.RPS = rounds_per_slice(G, b);
        E.NS = slices_of(G, b);
        E.units = G.Hkv * b.nblk;
        if ((int64_t)E.units * E.NS * E.RPS > kMaxRounds) return hipErrorInvalidValue;
        A.rounds += (unsigned)E.units * E.NS * E.RPS;
        slices += (int64_t)E.units * E.NS;
        alike = alike && E.RPS == A.e[0].RPS;
    }
    for (int i = count; i < kMaxWide; ++i) A.e[i] = A.e[0];
    const int64_t places = 2 * wide_cus();   // two workgroups per compute unit
    A.direct = count == 1 && slices <= places;
    const dim3 grid = A.direct ? dim3((unsigned)A.e[0].NS, (unsigned)b.nblk, (unsigned)G0.Hkv) : dim3((unsigned)std::min(slices, places));
    A.share = A.rounds / grid.x;         // (of a launch with a grid of one dimension)
    A.more = A.rounds % grid.x;
    A.reversed = !A.direct && alike && reverse_shares(A.rounds, grid.x, (unsigned)A.e[0].RPS);
    if (once) {
        const bool paged = G0.k_table != nullptr;
        if (!A.direct || b.ru != 8) return hipErrorInvalidValue;
        if (dtype == 0) return D == 128 ? launch_once<w_bf16, 128>(A, paged, grid, st) : launch_once<w_bf16, 64>(A, paged, grid, st);
        return D == 128 ? launch_once<w_f16, 128>(A, paged, grid, st) : launch_once<w_f16, 64>(A, paged, grid, st);
    }
    if (dtype == 0) return D == 128 ? by_rows<w_bf16, 128>(A, b.ru, grid, st) : by_rows<w_bf16, 64>(A, b.ru, grid, st);
    return D == 128 ? by_rows<w_f16, 128>(A, b.ru, grid, st) : by_rows<w_f16, 64>(A, b.ru, grid, st);
}

hipError_t launch_score_wide(int dtype, int D, int count, const WidePrompt* P, hipStream_t st, const WideClear& clear) {
    return score_wide(dtype, D, count, P, st, clear, false, nullptr);
}

int64_t wide_once_pairs(const ScoreGeom& G) {
    Blocks b;
    return wide_shape(G, &b) ? (int64_t)G.Hkv * b.nblk * slices_of(G, b) * b.ru * 16 : 0;
}

// A workgroup per slice, two per compute unit, and words that the hand-off region of the single-read kernel holds.
bool wide_once_ok(int dtype, int D, const ScoreGeom& G) {
    Blocks b;
    return wide_ok(dtype, D, G) && row_blocks(G, &b) && b.ru == 8 && (size_t)wide_once_pairs(G) * sizeof(float2) <= fused_sync_bytes(G) &&
           (int64_t)G.Hkv * b.nblk * slices_of(G, b) <= 2 * wide_cus();
}

hipError_t launch_score_wide_once(int dtype, int D, const WidePrompt& P, unsigned* gave_up, hipStream_t st) {
    return score_wide(dtype, D, 1, &P, st, WideClear{}, true, gave_up);
}

}  // namespace snapkv
