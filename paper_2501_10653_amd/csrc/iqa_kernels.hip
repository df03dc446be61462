// Tile-wise LISI / augLISI on gfx950: one fused streaming pass over both images.
//
// What is computed (Li, Adamek & Armour, Sec. 1-3): after the Sec. 2 clamp of
// negative pixels to zero, every N_T x N_T tile gets
//   A = sum (x'+y')/(|x'-y'|+C1),  P = sum (x'+y')|x'-y'|,  Sx = sum x',  Sy = sum y'
//   lisi = D*A/(max(Sx,Sy)+C2)  (Eq. 1),   auglisi = 1 - P/(Sx+Sy+C)  (Eq. 2).
//
// How (MI355X design, not the paper's block-per-tile shared-memory scheme):
//   * The work is HBM-bound: 8 bytes per pixel pair against ~18 VALU slots, so
//     the kernel's job is to keep enough 128-bit loads in flight and to spend
//     as few instructions as possible outside the per-pixel loop.
//   * A wave of 64 lanes is cut into groups of seg*rp lanes, one group per
//     tile, which read the tile's rows in 16-byte quads: short tile rows a few
//     at a time, long ones quad by quad in turn (see slice_sums).  So a wave
//     covers 64/(seg*rp) adjacent tiles, and a whole tile slice reduces inside
//     one wave with DPP lane permutations, with no LDS and no barrier.  Several
//     waves of a workgroup may share a tile's rows (combined once in LDS), and
//     for shapes with few large tiles several workgroups share them (the last
//     of them to finish combines their partials, chosen by an atomic ticket; no
//     second launch).
//   * Each lane folds up to 16 pixels with plain FP32 (FMA chains) and adds the
//     block into Kahan-compensated (hi, lo) accumulators: the long per-lane sums
//     are compensated.  Across lanes the partial sums are folded to one float
//     and added plainly: every partial is non-negative, so a tree of depth d
//     adds at most d units of roundoff, relative.
//   * Loads are double-buffered: the next `unroll` rows are in flight while the
//     current ones are reduced.
//   * Every reduction has a fixed order and there are no floating-point
//     atomics, so results are bitwise reproducible and bitwise symmetric in x, y.
//   * LISI's quotient and augLISI = 1 - P/S are finalised in double-float: the
//     one adds a single rounding, the other's subtraction keeps the accuracy of
//     the sums.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <type_traits>
#include <utility>
#include <vector>

#include "iqa.h"
#include "iqa_internal.h"

namespace iqa {

constexpr int kWave = 64;
enum Mode : int { kLisi = 1, kAug = 2, kBoth = 3 };
// How the parts of a split tile group are added up (see split_finish).
enum SplitMode : int { kSplitNone = 0, kSplitTicket = 1, kSplitCombine = 2 };

// One pair's work (also a batch descriptor's payload): see slice_sums for the
// geometry fields.
struct PairArgs {
    const float *x;
    const float *y;
    float *lisi;
    float *aug;
    float *sums;
    float D, C1, C2, C;
    int32_t N;           // image side (row stride in floats), <= 2^17
    int32_t NT;          // tile side
    int32_t ns;          // tiles per side
    int32_t ngx;         // tile groups along x: ceil(ns / ht)
    uint32_t ngx_m;      // division multiplier for ngx (see udiv)
    int32_t log_grp;     // log2(G), lanes per tile in a wave; ht = 64 / G tiles per wave
    int32_t rows_wave;   // tile rows per wave slice: NT / (waves * ks); ANY: per part, NT / ks
    int32_t cols;        // quads (VEC pixels) per tile row: ceil(NT / vec)
    int32_t pitch;       // quad places per tile row that the lanes count with
    uint32_t pitch_m;    // ceil(2^31 / pitch)
    int32_t lead;        // lead_rows * pitch - shift (these three: not ANY)
    int32_t lead_rows;   // rows above the slice that lane 0 starts counting from
    int32_t step;        // bytes from one of a lane's items to the next, before a wrap
    int64_t items;       // loads per lane and image: ceil(rows_wave * pitch / G)
};

struct KArgs : PairArgs {
    int32_t smode;       // split tiles: kSplitNone, kSplitTicket or kSplitCombine
    int32_t ks;          // workgroups per tile group
    uint32_t ks_m;       // division multiplier for ks
    float *ws;           // split partials: [group][ks][ht][4]
};

__host__ __device__ __forceinline__ int tiles_per_wave(const PairArgs &a) {
    return 64 >> a.log_grp;
}

// ---------------------------------------------------------------------------
// Compensated FP32 arithmetic
// ---------------------------------------------------------------------------

struct CSum {
    float hi, lo;   // value = hi + lo
};

// Kahan step: add v, keeping in lo what the rounding of hi lost.
__device__ __forceinline__ void cadd(CSum &a, float v) {
    const float y = v + a.lo;
    const float t = a.hi + y;
    a.lo = y - (t - a.hi);
    a.hi = t;
}

// Exact error-free sum s + e = a + b (Knuth's TwoSum; no ordering needed).
__device__ __forceinline__ void two_sum(float a, float b, float &s, float &e) {
    s = a + b;
    const float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// n / d for d > 0 (normal, finite): the hardware reciprocal estimate, then one
// correction with the exact residual n - q*d from an FMA.  Within one unit in
// the last place (almost always the correctly rounded quotient) in 4
// dependent operations; an IEEE division is a chain of about 15.
__device__ __forceinline__ float div_pos(float n, float d, float rd) {
    const float q = n * rd;
    return __builtin_fmaf(__builtin_fmaf(-q, d, n), rd, q);
}

struct Acc {
    CSum A, P, X, Y;
};

__device__ __forceinline__ Acc acc_zero() {
    return Acc{{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
}

// ---------------------------------------------------------------------------
// Lane permutations
// ---------------------------------------------------------------------------

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

// All-reduce steps inside aligned lane groups.  Within a row of 16 lanes the
// partner comes from a DPP permutation: quad swaps for strides 1 and 2, then
// half-row and row mirrors for 4 and 8 (once the smaller strides have made
// each half uniform, a mirror pairs every lane with the other half).  Across
// rows, gfx950's permlane swaps exchange whole rows (16) or half-waves (32).
template <int CTRL>
__device__ __forceinline__ void dpp_add(float &v) {
    v += dpp<CTRL>(v);
}

template <int W>
__device__ __forceinline__ void permlane_swap(float &a, float &b) {
    const auto r = W == 16 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(a),
                                                              __float_as_uint(b), false, false)
                           : __builtin_amdgcn_permlane32_swap(__float_as_uint(a),
                                                              __float_as_uint(b), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

// One swap level for a single value: with both operands equal, the two
// results are the two halves of a row pair (W = 16) or of the wave (W = 32),
// and their sum is the same on every lane.
template <int W>
__device__ __forceinline__ void swap_add(float &v) {
    float a = v, b = v;
    permlane_swap<W>(a, b);
    v = a + b;
}

// The same level for two values with two swaps instead of two pairs of
// swaps and adds.  Swapping between a and b leaves in one half of each row
// pair (or wave) a's two halves and in the other b's; one add then forms a's
// total in the first and b's in the second, with the operands in the order
// swap_add uses, so the bits are the same.  Swapping that sum with itself
// hands both totals to every lane.
template <int W>
__device__ __forceinline__ void swap_add2(float &a, float &b) {
    permlane_swap<W>(a, b);
    float t = a + b, u = t;
    permlane_swap<W>(t, u);
    a = t;
    b = u;
}

// Plain sums over aligned groups of 2^log_g lanes; every lane of a group ends
// with the same bits (each step adds the same two values).
struct Sum4 {
    float A, P, X, Y;
};

template <int MODE, typename Step>
__device__ __forceinline__ void each(Sum4 &s, Step step) {
    if constexpr ((MODE & kLisi) != 0) step(s.A);
    if constexpr ((MODE & kAug) != 0) step(s.P);
    step(s.X);
    step(s.Y);
}

template <int MODE, int W>
__device__ __forceinline__ void swap_level(Sum4 &s) {
    if constexpr (MODE == kBoth) {
        swap_add2<W>(s.A, s.P);
    } else if constexpr (MODE == kLisi) {
        swap_add<W>(s.A);
    } else {
        swap_add<W>(s.P);
    }
    swap_add2<W>(s.X, s.Y);
}

// log_g is uniform, so the level tests are scalar branches; marked likely,
// they keep the levels a group needs in one straight run of code.
template <int MODE>
__device__ __forceinline__ Sum4 group_allreduce(Sum4 s, int log_g) {
    if (__builtin_expect(log_g > 0, 1)) {
        each<MODE>(s, [](float &v) { dpp_add<0xB1>(v); });    // quad_perm [1,0,3,2]
        if (__builtin_expect(log_g > 1, 1)) {
            each<MODE>(s, [](float &v) { dpp_add<0x4E>(v); });    // quad_perm [2,3,0,1]
            if (__builtin_expect(log_g > 2, 1)) {
                each<MODE>(s, [](float &v) { dpp_add<0x141>(v); });   // row_half_mirror
                if (__builtin_expect(log_g > 3, 1)) {
                    each<MODE>(s, [](float &v) { dpp_add<0x140>(v); });   // row_mirror
                    if (__builtin_expect(log_g > 4, 1)) {
                        swap_level<MODE, 16>(s);
                        if (__builtin_expect(log_g > 5, 1)) swap_level<MODE, 32>(s);
                    }
                }
            }
        }
    }
    return s;
}

__device__ __forceinline__ Sum4 fold(const Acc &a) {
    return Sum4{a.A.hi + a.A.lo, a.P.hi + a.P.lo, a.X.hi + a.X.lo, a.Y.hi + a.Y.lo};
}

// The same steps for sums in FP64.
struct Sum4d {
    double A, P, X, Y;
};

template <int MODE, typename Step>
__device__ __forceinline__ void each(Sum4d &s, Step step) {
    if constexpr ((MODE & kLisi) != 0) step(s.A);
    if constexpr ((MODE & kAug) != 0) step(s.P);
    step(s.X);
    step(s.Y);
}

__device__ __forceinline__ double with_words(float hi, float lo) {
    return __hiloint2double(__float_as_int(hi), __float_as_int(lo));
}

template <int MODE, int CTRL>
__device__ __forceinline__ void lanes_add(Sum4d &s) {
    each<MODE>(s, [](double &v) {
        v += with_words(dpp<CTRL>(__int_as_float(__double2hiint(v))),
                        dpp<CTRL>(__int_as_float(__double2loint(v))));
    });
}

// ---------------------------------------------------------------------------
// Per-pixel work
// ---------------------------------------------------------------------------

template <int VEC> struct VecT;
template <> struct VecT<4> { using T = float4; };
template <> struct VecT<2> { using T = float2; };
template <> struct VecT<1> { using T = float; };

// Streaming loads: every input byte is read exactly once, so they carry the
// nontemporal hint and do not displace other data in the caches.
//
// The pointer is cast to the global address space: pointers that come out of a
// batch descriptor in memory are not known to be global, and a flat load
// checks the LDS aperture and counts on both wait counters.  ANY: a quad at any
// float address (the hardware takes a 16-byte global load at 4-byte alignment).
#define IQA_GLOBAL __attribute__((address_space(1)))
#define IQA_CONSTANT __attribute__((address_space(4)))

template <int VEC, bool ANY = false>
__device__ __forceinline__ typename VecT<VEC>::T vload(const IQA_GLOBAL char *p) {
    if constexpr (VEC == 4 && ANY) {
        typedef float f4 __attribute__((ext_vector_type(4), aligned(4)));
        const f4 v = __builtin_nontemporal_load(reinterpret_cast<const IQA_GLOBAL f4 *>(p));
        return float4{v.x, v.y, v.z, v.w};
    } else if constexpr (VEC == 4) {
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 v = __builtin_nontemporal_load(reinterpret_cast<const IQA_GLOBAL f4 *>(p));
        return float4{v.x, v.y, v.z, v.w};
    } else if constexpr (VEC == 2) {
        typedef float f2 __attribute__((ext_vector_type(2)));
        const f2 v = __builtin_nontemporal_load(reinterpret_cast<const IQA_GLOBAL f2 *>(p));
        return float2{v.x, v.y};
    } else {
        return __builtin_nontemporal_load(reinterpret_cast<const IQA_GLOBAL float *>(p));
    }
}

__device__ __forceinline__ const IQA_GLOBAL char *global_bytes(const float *p) {
    return reinterpret_cast<const IQA_GLOBAL char *>(reinterpret_cast<uintptr_t>(p));
}

template <int VEC>
__device__ __forceinline__ typename VecT<VEC>::T vzero() {
    typename VecT<VEC>::T z;
    std::memset(&z, 0, sizeof(z));
    return z;
}

template <int VEC>
__device__ __forceinline__ float velem(const typename VecT<VEC>::T &v, int e) {
    if constexpr (VEC == 1) {
        return v;
    } else {
        return reinterpret_cast<const float *>(&v)[e];
    }
}

// Per-pixel terms of VEC adjacent pixel pairs, added to a short block sum b in
// plain FP32: products as FMA chains, the four pixels of a quad in pairs first.  A
// pair of zeros adds nothing.  SKIP: the first `skip` elements are not counted
// (the clamp's threshold is infinite).
template <int VEC, int MODE, bool SKIP = false>
__device__ __forceinline__ void accumulate(const typename VecT<VEC>::T &xv,
                                           const typename VecT<VEC>::T &yv, float C1, Sum4 &b,
                                           int skip = 0) {
    float xc[VEC], yc[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const float xr = velem<VEC>(xv, e);
        const float yr = velem<VEC>(yv, e);
        const float floor = SKIP && e < skip ? __builtin_inff() : 0.f;
        xc[e] = xr > floor ? xr : 0.f;   // Sec. 2 clamp; NaN and -0 -> +0
        yc[e] = yr > floor ? yr : 0.f;
        const float s = xc[e] + yc[e];          // |x'+y'| (both non-negative)
        const float d = fabsf(xc[e] - yc[e]);   // |x'-y'|
        if constexpr ((MODE & kLisi) != 0) {
            const float r = __builtin_amdgcn_rcpf(d + C1);
            b.A = __builtin_fmaf(s, r, b.A);
        }
        if constexpr ((MODE & kAug) != 0) b.P = __builtin_fmaf(s, d, b.P);
    }
    if constexpr (VEC == 4) {
        b.X += (xc[0] + xc[1]) + (xc[2] + xc[3]);
        b.Y += (yc[0] + yc[1]) + (yc[2] + yc[3]);
    } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            b.X += xc[e];
            b.Y += yc[e];
        }
    }
}

// Add a block sum into the Kahan-compensated lane accumulators.
template <int MODE>
__device__ __forceinline__ void add_block(Acc &acc, const Sum4 &b) {
    if constexpr ((MODE & kLisi) != 0) cadd(acc.A, b.A);
    if constexpr ((MODE & kAug) != 0) cadd(acc.P, b.P);
    cadd(acc.X, b.X);
    cadd(acc.Y, b.Y);
}

// ---------------------------------------------------------------------------
// Finalisation (Eq. 1, Eq. 2)
// ---------------------------------------------------------------------------

// A tile's sums reach these as plain FP32 values: each lane folded its
// compensation in before the cross-lane adds.

// Eq. 1, with the roundings of the numerator and the denominator corrected in the
// quotient (as plain FP32 operations they were most of LISI's error: 2048^2/64 rms
// 1.19 units of roundoff, 1.06 so).
__device__ __forceinline__ void finalize_lisi(const PairArgs &a, int64_t t, const Sum4 &s) {
    if (!a.lisi) return;
    float d, dl;
    two_sum(fmaxf(s.X, s.Y), a.C2, d, dl);
    const float n = a.D * s.A;
    const float nl = __builtin_fmaf(a.D, s.A, -n);
    const float rd = __builtin_amdgcn_rcpf(d);
    const float q = n * rd;
    float r = __builtin_fmaf(-q, d, n);   // remainder of (n + nl) / (d + dl)
    r += __builtin_fmaf(-q, dl, nl);
    a.lisi[t] = __builtin_fmaf(r, rd, q);
}

// Eq. 2: S = Sx + Sy + C and q = P / S in double-float, then 1 - q.
__device__ __forceinline__ void finalize_aug(const PairArgs &a, int64_t t, const Sum4 &s) {
    if (!a.aug) return;
    float s1, e1;
    two_sum(s.X, s.Y, s1, e1);
    float s2, e2;
    two_sum(s1, a.C, s2, e2);
    float Sh, Sl;
    two_sum(s2, e1 + e2, Sh, Sl);
    const float rS = __builtin_amdgcn_rcpf(Sh);
    const float q1 = div_pos(s.P, Sh, rS);
    float r = __builtin_fmaf(-q1, Sh, s.P);    // remainder of P / Sh
    r = __builtin_fmaf(-q1, Sl, r);
    const float q2 = r * rS;                   // correction term: a few bits suffice
    float h, e;
    two_sum(1.0f, -q1, h, e);
    a.aug[t] = h + (e - q2);
}

__device__ __forceinline__ void store_sums(const PairArgs &a, int64_t t, const Sum4 &s) {
    if (a.sums) reinterpret_cast<float4 *>(a.sums)[t] = float4{s.A, s.P, s.X, s.Y};
}

template <int MODE>
__device__ __forceinline__ void finalize(const PairArgs &a, int64_t t, const Sum4 &s) {
    if constexpr ((MODE & kLisi) != 0) finalize_lisi(a, t, s);
    if constexpr ((MODE & kAug) != 0) finalize_aug(a, t, s);
    if constexpr (MODE == kBoth) store_sums(a, t, s);
}

// The dispatcher hands workgroup b to XCD b % 8, and each XCD has its own L2
// whose channels interleave on low address bits.  Renumbering so that XCD x
// gets one contiguous range of logical workgroups keeps every XCD streaming
// from all column offsets (and so from all of its L2 channels) instead of the
// one offset class that b % 8 would give it.
constexpr int kLogXcds = 3, kXcds = 1 << kLogXcds;

__device__ __forceinline__ int xcd_remap(uint32_t b, uint32_t grid) {
    const uint32_t xcd = b % kXcds;
    const uint32_t local = b / kXcds;
    const uint32_t full = grid / kXcds;
    const uint32_t rem = grid % kXcds;
    return (int)(xcd * full + (xcd < rem ? xcd : rem) + local);
}

// Division by a divisor d fixed for the launch (1 <= d < 2^31), for numerators
// 0 <= n < 2^31, without the ~30-instruction integer division sequence: with
// l = ceil(log2 d) and m = floor(2^(31+l) / d) + 1 (< 2^32, computed on the
// host by div_magic), n / d = (n * m) >> (31 + l) exactly (Granlund and
// Montgomery, "Division by invariant integers using multiplication", 1994,
// Theorem 4.2 with 31-bit numerators).  Block indices are wave-uniform, so
// this runs on the scalar unit ahead of the first load.
__device__ __forceinline__ int udiv(int n, uint32_t m, int d) {
    const uint32_t l = d > 1 ? 32u - (uint32_t)__clz((uint32_t)d - 1u) : 0u;
    return (int)(((uint64_t)(uint32_t)n * m) >> (31u + l));
}

// ---------------------------------------------------------------------------
// Timeline stamps (diagnostic launches only)
// ---------------------------------------------------------------------------
//
// The constant-rate wall clock, read once `v` has been computed: the empty
// volatile asm needs v in a register, and volatile statements keep their
// order with the clock read, so the stamp cannot move above the arithmetic
// (and the loads) that produced v.
__device__ __forceinline__ uint64_t stamp_after(float v) {
    asm volatile("" ::"v"(v));
    return wall_clock64();
}

// ---------------------------------------------------------------------------
// One wave's slice of one tile group
// ---------------------------------------------------------------------------
//
// A tile group is the ht = 64/G horizontally adjacent tiles one wave covers:
// tiles txg*ht .. txg*ht+ht-1 of tile row ty.  A slice is rows
// slice*rows_wave .. (slice+1)*rows_wave-1 of those tiles.  Lane L belongs to
// tile j = L / G of the group.  A tile row is `cols` quads of VEC pixels, on
// `pitch` places; the tile's part of the slice is rows_wave * pitch places
// counted row by row, and the G lanes of a tile take them in turn: lane q has
// places q - shift, q - shift + G, ..., with shift chosen so that the last item
// of every lane exists and only the first may fall before the slice.  Returns
// the slice's sums of tile j, the same on every lane of the tile's lane group.
//
// Rows of at most G quads have a pitch of the next power of two: a lane keeps
// its column (lanes past `cols` idle) and takes every (G/pitch)-th row, at a
// constant 32-bit step from scalar bases (a slice spans at most 256 rows, below
// 2^28 bytes).  WRAP, longer rows: pitch == cols, so all lanes always work; a
// lane moves G quads on from item to item, and to the next row where that
// leaves its row.  (Counting short rows without gaps too keeps every lane busy
// but cuts each load instruction into more pieces: measured on a mix of tile
// sides from 12 to 100, 2 to 17% slower, e.g. 2000^2/50 9.2 against 7.9 us.
// For wide rows it is what keeps a 300-pixel row, 75 quads, from taking two
// loads: 3000^2/300 15.7 against 17.0 us.)
//
// Items are read in batches of U with the next batch in flight while the
// current one is reduced, in blocks of kBlock items of plain FP32 sums between
// two compensated additions.  Items beyond a multiple of U form a batch of their
// own that goes first, so every load has others in flight with it; the item that
// some lanes lack is always in it.  It is often all that a lane has, and is
// reduced in blocks of two.  (Compensating every item costs 1.5% at 2025^2/45 and
// 3000^2/100; blocks of eight, 32 pixels, raise the rms error of the sums at
// 8192^2/16 from 0.72 units of roundoff to 0.84.)
//
// ANY (VEC 4): images at any float address and any NT >= 4.  A lane loads a
// quad wherever it lies; the last quad of a tile row is moved back to end with
// the row, and the pixels it then shares with its neighbour are not counted.
// NT may be odd, so the slices are quarters of a part's rows, uneven by a row,
// and their items are counted here.  (One wave per part against four, each with
// its best lanes per tile, in us: 2025^2/45 9.1 and 8.4, 8190^2/90 92.5 and
// 85.8, 500^2/50 5.0 and 4.0, 1000^2/250 6.2 and 5.5; 2000^2/50 8.1 both;
// 2025^2/25 7.6 and 8.3, 3000^2/75 15.4 and 16.1.  Two waves lie between.)
constexpr int kAnyWaves = 4;
constexpr int kBlock = 4;

template <int VEC, bool ANY, int U, int MODE, bool WRAP, bool TL = false>
__device__ __forceinline__ Sum4 slice_sums(const PairArgs &a, int ty, int txg, int slice, int lane,
                                           uint64_t *ts = nullptr) {
    using V = typename VecT<VEC>::T;
    const int G = 1 << a.log_grp;
    const int q = lane & (G - 1);
    const int tx0 = txg * tiles_per_wave(a);
    const int j = lane >> a.log_grp;

    Acc acc = acc_zero();
    int slice_row, lead, lead_rows;
    int64_t items;
    if constexpr (ANY) {
        const int part = slice / kAnyWaves, w = slice % kAnyWaves;
        const int from = w * a.rows_wave / kAnyWaves;
        const int rows = (w + 1) * a.rows_wave / kAnyWaves - from;
        slice_row = part * a.rows_wave + from;
        if constexpr (WRAP) {   // shift < G < cols
            const int64_t places = (int64_t)rows * a.cols;
            items = (places + G - 1) >> a.log_grp;
            const int shift = (int)((items << a.log_grp) - places);
            lead_rows = shift ? 1 : 0;
            lead = shift ? a.cols - shift : 0;
        } else {                // whole rows: G / pitch at a time
            const int log_rows = a.log_grp - __builtin_ctz(a.pitch);
            items = (rows + (1 << log_rows) - 1) >> log_rows;
            lead_rows = (int)(items << log_rows) - rows;
            lead = 0;
        }
    } else {
        slice_row = slice * a.rows_wave;
        items = a.items;
        lead = a.lead;
        lead_rows = a.lead_rows;
    }
    // Row and column of the lane's first item, counted from lead_rows above
    // the slice (f * pitch < 2^31: the quotient is exact).
    const uint32_t f = (uint32_t)(q + lead);
    const int r = (int)__umulhi(f << 1, a.pitch_m);
    int col = (int)f - r * a.pitch;
    if (tx0 + j < a.ns && (WRAP || col < a.cols)) {
        const int shift = lead_rows * a.pitch - lead;
        const bool has_first = q >= shift;
        // The slice's first pixel, at most 2^17 rows of at most 2^17 pixels
        // down; the bases of lanes without a first item may lie above the image.
        const uint32_t row0 = (uint32_t)(ty * a.NT + slice_row);
        const uint64_t first = (uint64_t)row0 * (uint32_t)a.N + (uint32_t)(tx0 * a.NT);
        const int64_t base = (int64_t)first * 4 - (int64_t)((uint32_t)(lead_rows * a.N) * 4u);
        const IQA_GLOBAL char *bx = global_bytes(a.x) + base;
        const IQA_GLOBAL char *by = global_bytes(a.y) + base;
        const int over = a.cols * VEC - a.NT;   // ANY: pixels the last quad moves back
        uint32_t off = (uint32_t)(r * a.N + j * a.NT + col * VEC) * 4u;
        int skip = 0;                          // ANY without WRAP: pixels not counted
        if constexpr (ANY && !WRAP) {
            skip = col == a.cols - 1 ? over : 0;
            off -= (uint32_t)skip * 4u;
        }
        if constexpr (WRAP) {   // the lanes move apart: per-lane addresses
            bx += off;
            by += off;
            off = 0;
        }
        const int64_t wrap_step = (int64_t)a.step + (int64_t)a.N * 4 - (int64_t)a.cols * (VEC * 4);
        auto load_item = [&](V &xv, V &yv, bool ok, int u, uint32_t &last) {
            int back = 0;
            if constexpr (ANY && WRAP) {
                const bool end = col == a.cols - 1;
                back = end ? over * 4 : 0;
                last |= end ? 1u << u : 0u;
            }
            if (ok) {
                xv = vload<VEC, ANY>(bx + off - back);
                yv = vload<VEC, ANY>(by + off - back);
            } else {
                xv = vzero<VEC>();
                yv = vzero<VEC>();
            }
            if constexpr (WRAP) {
                col += G;
                const bool wrap = col >= a.cols;
                col -= wrap ? a.cols : 0;
                bx += wrap ? wrap_step : a.step;
                by += wrap ? wrap_step : a.step;
            } else {
                off += (uint32_t)a.step;
            }
        };
        auto load = [&](V (&xv)[U], V (&yv)[U], uint32_t &last) {
            last = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) load_item(xv[u], yv[u], true, u, last);
        };
        auto quad = [&](const V (&xv)[U], const V (&yv)[U], uint32_t last, int u, Sum4 &b) {
            int sk = skip;
            if constexpr (ANY && WRAP) sk = (last >> u) & 1 ? over : 0;
            accumulate<VEC, MODE, ANY>(xv[u], yv[u], a.C1, b, sk);
        };
        auto reduce = [&](const V (&xv)[U], const V (&yv)[U], uint32_t last) {
#pragma unroll
            for (int u = 0; u < U; u += kBlock) {
                Sum4 b{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int v = u; v < u + kBlock; ++v) quad(xv, yv, last, v, b);
                add_block<MODE>(acc, b);
            }
        };
        // Full batches, and the items of the partial one (0..U).
        using Count = std::conditional_t<WRAP, uint64_t, uint32_t>;
        const Count n = (Count)items;
        Count left = (n - (shift ? 1 : 0)) / U;
        const int part = (int)(n - left * U);

        V ax[U], ay[U], cx[U], cy[U];
        uint32_t alast = 0, clast = 0;
        if (part) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (u < part) load_item(cx[u], cy[u], u > 0 || has_first, u, clast);
        }
        if (left) load(ax, ay, alast);
        if (part) {
#pragma unroll
            for (int u = 0; u < U; u += 2) {
                if (u >= part) break;
                Sum4 b{0.f, 0.f, 0.f, 0.f};
                quad(cx, cy, clast, u, b);
                if (u + 1 < part) quad(cx, cy, clast, u + 1, b);
                if (u == 0) {   // what add_block makes of zero
                    acc = Acc{{b.A, 0.f}, {b.P, 0.f}, {b.X, 0.f}, {b.Y, 0.f}};
                } else {
                    add_block<MODE>(acc, b);
                }
            }
            if constexpr (TL) ts[0] = stamp_after(acc.X.hi);
        }
        if (left) {
            while (true) {
                const bool more_c = left > 1;
                if (more_c) load(cx, cy, clast);
                reduce(ax, ay, alast);
                if constexpr (TL) {
                    if (ts[0] == 0) ts[0] = stamp_after(acc.X.hi);
                }
                if (!more_c) break;
                const bool more_a = left > 2;
                if (more_a) load(ax, ay, alast);
                reduce(cx, cy, clast);
                if (!more_a) break;
                left -= 2;
            }
        }
    }
    if constexpr (TL) ts[1] = stamp_after(acc.X.hi);

    // Sum the lanes of each tile inside the wave.
    return group_allreduce<MODE>(fold(acc), a.log_grp);
}

// Pairwise tree over the partial sums of WAVES waves (all non-negative), in a
// fixed order: the same bits wherever a tile's slices are combined.
template <int WAVES>
__device__ __forceinline__ float4 wave_tree(float4 (&v)[WAVES]) {
#pragma unroll
    for (int h = 1; h < WAVES; h *= 2) {
#pragma unroll
        for (int w = 0; w + h < WAVES; w += 2 * h) {
            v[w].x += v[w + h].x;
            v[w].y += v[w + h].y;
            v[w].z += v[w + h].z;
            v[w].w += v[w + h].w;
        }
    }
    return v[0];
}

// One wave finishes the tiles of a group from the waves' sums in LDS, lane j tile
// j.  Quads at any address and the smallest tiles have more waves on a tile than
// compensation alone would ask for, so their sums are added without further
// roundoff: a quad of lanes per tile, one of the four sums each, in FP64 (2025^2/45:
// rms errors of P and Sx 0.82 and 0.71 units of roundoff as a tree, 0.68 and 0.60
// so, and 0.1 us of 8.2; 2024^2/8 A 0.79 and 0.68, and 0.3 us of 7.3).
template <bool ANY, int WAVES, typename Finish>
__device__ __forceinline__ void finish_group(const PairArgs &a, const float4 (&lds)[WAVES][kWave],
                                             int ty, int txg, int lane, Finish finish) {
    const int ht = tiles_per_wave(a);
    if (ANY || a.log_grp <= 2) {
        for (int j0 = 0; j0 < ht; j0 += kWave / 4) {
            const int j = j0 + (lane >> 2), tx = txg * ht + j;
            const bool mine = j < ht && tx < a.ns;
            double v = 0.0;
            if (mine) {
                const float *w = reinterpret_cast<const float *>(&lds[0][j]) + (lane & 3);
#pragma unroll
                for (int i = 0; i < WAVES; ++i) v += (double)w[i * kWave * 4];
            }
            const float s = (float)v;
            const Sum4 r{s, dpp<0x55>(s), dpp<0xAA>(s), dpp<0xFF>(s)};   // of the quad's lanes
            if (mine && (lane & 3) == 0) finish((int64_t)ty * a.ns + tx, r);
        }
    } else {
        const int tx = txg * ht + lane;
        if (lane >= ht || tx >= a.ns) return;
        float4 w[WAVES];
#pragma unroll
        for (int i = 0; i < WAVES; ++i) w[i] = lds[i][lane];
        const float4 v = wave_tree<WAVES>(w);
        finish((int64_t)ty * a.ns + tx, Sum4{v.x, v.y, v.z, v.w});
    }
}

// ---------------------------------------------------------------------------
// Split tiles: adding up the parts of a tile group
// ---------------------------------------------------------------------------
//
// With ks > 1 workgroups per tile group, every part stores its partial sums
// (one float4 per tile), and the parts are added in one of two ways:
//
//   * kSplitTicket: each part then takes a ticket from the group's counter,
//     and the part that draws the last one adds the partials and finalises,
//     within the same launch; it also sets the counter back to zero.  No part
//     waits for another.  The parts run on different XCDs, whose L2 caches
//     are not coherent with one another, so the partials travel by
//     device-coherent accesses (agent-scope atomic stores and loads, which
//     bypass the non-coherent cache levels), and only the ordering is left to
//     the counter: a part's partial stores have completed (vmcnt 0) before it
//     takes its ticket, and the last part issues its partial loads only after
//     its ticket has returned.
//   * kSplitCombine: the parts only store their partials, and combine_kernel,
//     launched right after on the same stream, adds them.
//
// The ticket costs every part a few memory round trips at its end (store
// acknowledgement, atomic); while a launch fits the GPU in one round of
// workgroups that is cheaper than a second launch, but when many rounds of
// workgroups queue behind those round trips it is not, and the host picks
// the combine launch (split_mode).
//
// Either way the partials are added the way the kernel adds pixels: a lane of
// tile j's lane group adds every so many of them with compensation, then the
// group is summed with the same fixed DPP tree (parts_sum).  The order depends
// neither on the mechanism nor on which part came last, so results are bitwise
// reproducible and equal between the two.
//
// Workspace: partials [group][part][ht] float4 from a.ws on, and (ticket
// mode) one 32-bit counter per group below a.ws (group g's at
// a.ws - kLine (g + 1) bytes), in a counter region that holds nothing but
// counters.  The counters start at zero and every launch leaves the ones it
// used at zero, so a region reused by shapes of any size is all zeros between
// launches.  In ticket mode the parts' partials and the counters of different
// groups lie on lines of their own: coherent accesses of different XCDs to one
// line go one after the other.  (With 16-byte partials and 4-byte counters
// side by side a ticket launch paid about 10 ns per workgroup: 1000^2/250 in 50
// parts 14.0 us against 6.1, 2048^2/512 in 16 parts of sixteen waves 10.9
// against 9.1.)
constexpr int64_t kLine = 128;

__host__ __device__ __forceinline__ int64_t part_entries(int smode, int64_t ht) {
    return smode == kSplitTicket && ht * 16 < kLine ? kLine / 16 : ht;   // float4 per part
}

__device__ __forceinline__ void store_coherent(float4 *p, float4 v) {
    uint64_t *q = reinterpret_cast<uint64_t *>(p);
    const uint64_t lo = (uint64_t)__float_as_uint(v.x) | ((uint64_t)__float_as_uint(v.y) << 32);
    const uint64_t hi = (uint64_t)__float_as_uint(v.z) | ((uint64_t)__float_as_uint(v.w) << 32);
    __hip_atomic_store(q, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ float4 load_coherent(const float4 *p) {
    const uint64_t *q = reinterpret_cast<const uint64_t *>(p);
    const uint64_t lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return float4{__uint_as_float((uint32_t)lo), __uint_as_float((uint32_t)(lo >> 32)),
                  __uint_as_float((uint32_t)hi), __uint_as_float((uint32_t)(hi >> 32))};
}

// Wait until this wave's vector memory operations have completed.
__device__ __forceinline__ void wait_vmem() {
    __builtin_amdgcn_s_waitcnt(/*vmcnt*/ 0 | (/*expcnt*/ 0x7 << 4) | (/*lgkmcnt*/ 0xf << 8));
}

// Add up n parts of a tile, part(p), over its 2^log_g lanes (q: the lane's place
// among them); the first of them ends with the sums.  A power of two of parts:
// lane q has parts q, q + lanes, ..., and the lanes' tree is even.  Else that tree
// would be lopsided, and its error that of up to log2(n) additions of nearly the
// whole: a quarter to a half as many lanes, two to four parts each.  Up to sixteen
// parts are added in FP64, because the parts' own waves have left roundoff too
// (3000^2/300 in five parts: rms error of Sx 0.75 units of roundoff as a plain
// tree, 0.58 so, 0.69 in one workgroup; sixteen or more FP64 parts are too slow:
// 1536^2/768 in 96 parts 7.4 us as a plain tree, 7.9 in FP64, 7.4 compensated).
constexpr int kExactParts = 16;

template <int MODE, typename Part>
__device__ __forceinline__ Sum4 parts_sum(int n, int log_g, int q, Part part) {
    const int log_n = 31 - __clz(n);
    const bool even = n == 1 << log_n;
    const int log_l = min(log_g, even ? log_n : log_n - 1), lanes = 1 << log_l;
    const bool exact = !even && n < kExactParts;
    Acc c = acc_zero();
    Sum4d d{0.0, 0.0, 0.0, 0.0};
    for (int from = q; q < lanes && from < n; from += 4 * lanes) {
        float4 w[4];   // loads in flight, none behind a branch that would wait for one
#pragma unroll
        for (int i = 0; i < 4; ++i) w[i] = part(min(from + i * lanes, n - 1));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (from + i * lanes >= n) break;
            if (exact) {
                if constexpr ((MODE & kLisi) != 0) d.A += w[i].x;
                if constexpr ((MODE & kAug) != 0) d.P += w[i].y;
                d.X += w[i].z;
                d.Y += w[i].w;
            } else {
                if constexpr ((MODE & kLisi) != 0) cadd(c.A, w[i].x);
                if constexpr ((MODE & kAug) != 0) cadd(c.P, w[i].y);
                cadd(c.X, w[i].z);
                cadd(c.Y, w[i].w);
            }
        }
    }
    if (!exact) return group_allreduce<MODE>(fold(c), log_l);
    if (log_l > 0) lanes_add<MODE, 0xB1>(d);   // at most four lanes
    if (log_l > 1) lanes_add<MODE, 0x4E>(d);
    return Sum4{(float)d.A, (float)d.P, (float)d.X, (float)d.Y};
}

// Add up tile group grp's parts and finalise its tiles (one wave).  COHERENT
// reads the partials with device-coherent loads (within the launch that wrote
// them), else with plain loads (a later launch).
template <int MODE, bool COHERENT>
__device__ __forceinline__ void combine_parts(const KArgs &a, int grp, int lane) {
    const float4 *ws = reinterpret_cast<const float4 *>(a.ws);
    const int64_t base = (int64_t)grp * a.ks;
    const int64_t pitch = part_entries(a.smode, tiles_per_wave(a));
    const int ty = udiv(grp, a.ngx_m, a.ngx);
    const int txg = grp - ty * a.ngx;
    const int j = lane >> a.log_grp;   // the lane group's tile
    const int q = lane & ((1 << a.log_grp) - 1);
    const int tx = txg * tiles_per_wave(a) + j;
    // (A tile past the image's last has places for its parts too; its sums go nowhere.)
    const Sum4 s = parts_sum<MODE>(a.ks, a.log_grp, q, [&](int p) {
        const float4 *src = ws + (base + p) * pitch + j;
        return COHERENT ? load_coherent(src) : *src;
    });
    if (q == 0 && tx < a.ns) finalize<MODE>(a, (int64_t)ty * a.ns + tx, s);
}

// A part's end of a split tile group; returns whether this workgroup
// finished the group (ticket mode, last part).
template <int MODE>
__device__ __forceinline__ bool split_finish(const KArgs &a, int grp, int part, int lane, bool mine,
                                             int jt, float4 v) {
    float4 *ws = reinterpret_cast<float4 *>(a.ws);
    float4 *slot =
        ws + ((int64_t)grp * a.ks + part) * part_entries(a.smode, tiles_per_wave(a)) + jt;
    if (a.smode == kSplitCombine) {
        if (mine) *slot = v;
        return false;
    }
    if (mine) store_coherent(slot, v);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(a.ws) - (kLine / 4) * ((int64_t)grp + 1);
    wait_vmem();                                        // partials stored before the ticket
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    uint32_t ticket = 0;
    if (lane == 0) ticket = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ticket = __builtin_amdgcn_readfirstlane(ticket);    // waits for the returned value
    if (ticket != (uint32_t)(a.ks - 1)) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    combine_parts<MODE, true>(a, grp, lane);
    if (lane == 0) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
}

// ---------------------------------------------------------------------------
// The tile kernel (one image pair)
// ---------------------------------------------------------------------------
//
// Grid: one workgroup of WAVES waves per (tile group, split part).  The tile
// rows are cut into WAVES*ks contiguous slices of rows_wave rows; wave w of
// part p takes slice p*WAVES + w.
//
// SPLIT kernels (ks > 1 workgroups per tile group) finish through
// split_finish; the others finalise directly, and carry no split code.
//
// With several waves and both indices wanted, a workgroup that is not split
// finishes its tiles on two waves at once: wave 0 Eq. 1 (and the sums), wave
// 1 Eq. 2, each from the same LDS tree.
//
// TL (diagnostic launches only) records, per workgroup, wall-clock stamps of
// wave 0: entry, its first batch of rows reduced (first loads back), its last
// rows reduced (last loads back), and its exit after its results are stored,
// plus the XCD and hardware slot it ran on: 8 uint64 per workgroup at
// tl[8 * blockIdx.x], written with ordinary vector stores; the split part's
// word has bit 32 set when this workgroup finished its tiles.
template <int VEC, bool ANY, int WAVES, int U, int MODE, bool WRAP, bool SPLIT, bool TL>
__device__ __forceinline__ void tiles_body(const KArgs &a, uint64_t *tl) {
    uint64_t ts[4] = {0, 0, 0, 0};
    if constexpr (TL) ts[0] = wall_clock64();
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int bid = xcd_remap(blockIdx.x, gridDim.x);
    const int grp = udiv(bid, a.ks_m, a.ks);
    const int part = bid - grp * a.ks;
    const int ty = udiv(grp, a.ngx_m, a.ngx);
    const int txg = grp - ty * a.ngx;
    const int ht = tiles_per_wave(a);

    const Sum4 s = slice_sums<VEC, ANY, U, MODE, WRAP, TL>(a, ty, txg, part * WAVES + wave, lane, ts + 1);
    constexpr bool kTwoWaveFinish = WAVES > 1 && MODE == kBoth && !SPLIT;

    float4 v{s.A, s.P, s.X, s.Y};
    bool last = true;   // this workgroup finished its tiles
    if constexpr (WAVES == 1) {
        // A lane group's leader has its tile's sums.
        const int jt = lane >> a.log_grp;
        const bool mine = (lane & ((1 << a.log_grp) - 1)) == 0 && txg * ht + jt < a.ns;
        if constexpr (SPLIT) {
            last = split_finish<MODE>(a, grp, part, lane, mine, jt, v);
        } else {
            if (mine) finalize<MODE>(a, (int64_t)ty * a.ns + txg * ht + jt, s);
        }
    } else {
        // Combine the waves' slices of each tile in LDS, wave order fixed.
        __shared__ float4 lds[WAVES][kWave];
        if ((lane & ((1 << a.log_grp) - 1)) == 0) lds[wave][lane >> a.log_grp] = v;
        __syncthreads();
        if (wave != 0 && !(kTwoWaveFinish && wave == 1)) return;
        if constexpr (SPLIT) {
            const bool mine = lane < ht && txg * ht + lane < a.ns;
            if (mine) {
                float4 w[WAVES];
#pragma unroll
                for (int i = 0; i < WAVES; ++i) w[i] = lds[i][lane];
                v = wave_tree<WAVES>(w);
            }
            last = split_finish<MODE>(a, grp, part, lane, mine, lane, v);
        } else {
            finish_group<ANY>(a, lds, ty, txg, lane, [&](int64_t t, const Sum4 &r) {
                if constexpr (!kTwoWaveFinish) {
                    finalize<MODE>(a, t, r);
                } else if (wave == 0) {
                    finalize_lisi(a, t, r);
                    store_sums(a, t, r);
                } else {
                    finalize_aug(a, t, r);
                }
            });
        }
    }
    if constexpr (TL) {
        if (wave == 0) {
            __builtin_amdgcn_s_waitcnt(0);   // every store of the wave has landed
            const uint64_t t_end = wall_clock64();
            if (lane == 0) {
                uint64_t *r = tl + (int64_t)blockIdx.x * 8;
                r[0] = ts[0];
                r[1] = ts[1];
                r[2] = ts[2];
                r[3] = t_end;
                r[4] = (uint64_t)__builtin_amdgcn_s_getreg((31 << 11) | 20);   // XCC_ID
                r[5] = (uint64_t)__builtin_amdgcn_s_getreg((31 << 11) | 4);    // HW_ID
                r[6] = (uint64_t)grp;
                r[7] = (uint64_t)part | ((uint64_t)last << 32);
            }
        }
    }
}

// Batches of four leave room for five waves per SIMD, which small tiles need (at
// four, 3260^2/10 takes 18.3 us, and 16.3 with five); where the loop needs more
// registers than that (ANY with WRAP or SPLIT) they would go to memory.
template <int VEC, bool ANY, int WAVES, int U, int MODE, bool WRAP, bool SPLIT>
__global__ __launch_bounds__(WAVES * kWave, U == 4 && !(ANY && (WRAP || SPLIT)) ? 5 : 1) void
tiles_kernel(KArgs a) {
    tiles_body<VEC, ANY, WAVES, U, MODE, WRAP, SPLIT, false>(a, nullptr);
}

template <int VEC, int WAVES, int U, bool WRAP, bool SPLIT>
__global__ __launch_bounds__(WAVES * kWave) void tiles_kernel_tl(KArgs a, uint64_t *tl) {
    tiles_body<VEC, false, WAVES, U, kBoth, WRAP, SPLIT, true>(a, tl);
}

// A split launch without a workspace: one workgroup per tile (ht == 1) takes
// all of the tile's waves * ks slices, sixteen waves at a time, keeps their
// sums in LDS and adds them as the split launch does (the waves of each part by
// the same tree, the parts as combine_parts), so the bits are the same.  A part's
// slices are added by a thread each, all parts at once (within the last wave's
// loop over the parts, four reads per part one after the other, 400^2/200 took
// 10.6 us instead of 10.3, 900^2/300 20.6 instead of 20.4).
constexpr int kLocalWaves = 16;

template <bool ANY, int U, int MODE, bool WRAP>
__global__ __launch_bounds__(kLocalWaves * kWave) void tiles_local_kernel(KArgs a, int waves) {
    extern __shared__ float4 slices[];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int grp = xcd_remap(blockIdx.x, gridDim.x);
    const int ty = udiv(grp, a.ngx_m, a.ngx);
    const int tx = grp - ty * a.ngx;
    for (int i = wave; i < waves * a.ks; i += kLocalWaves) {
        const Sum4 s = slice_sums<4, ANY, U, MODE, WRAP>(a, ty, tx, i, lane);
        if (lane == 0) slices[i] = float4{s.A, s.P, s.X, s.Y};
    }
    __syncthreads();
    if (waves > 1) {   // each part's slices, as the tile kernel's waves are added
        for (int p = threadIdx.x; p < a.ks; p += kLocalWaves * kWave) {
            float4 *v = slices + p * waves;
            if (waves == 4) {
                float4 w[4] = {v[0], v[1], v[2], v[3]};
                v[0] = wave_tree<4>(w);
            } else {
                float4 w[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) w[i] = v[i];
                v[0] = wave_tree<8>(w);
            }
        }
        __syncthreads();
    }
    if (wave != 0) return;
    const Sum4 s = parts_sum<MODE>(a.ks, 6, lane, [&](int p) { return slices[p * waves]; });
    if (lane == 0) finalize<MODE>(a, (int64_t)ty * a.ns + tx, s);
}

// kSplitCombine: one wave per tile group adds its parts, after the tile
// kernel on the same stream (so the partials are complete and visible).
template <int MODE>
__global__ __launch_bounds__(kWave) void combine_kernel(KArgs a) {
    combine_parts<MODE, false>(a, (int)blockIdx.x, (int)threadIdx.x);
}

// ---------------------------------------------------------------------------
// The batched kernel (many image pairs of mixed N and N_T, one launch)
// ---------------------------------------------------------------------------
//
// Each pair is described by its own geometry and by the index of its first
// work unit.  A unit is the work of one workgroup of kBatchWaves waves:
//   * a pair whose geometry has one wave per tile group (waves 1) packs
//     kBatchWaves consecutive tile groups into a unit, wave w taking the
//     unit's w-th group;
//   * a pair whose geometry has kBatchWaves waves per tile group gives each
//     tile group a unit of its own: the waves take its row slices and combine
//     them in LDS exactly as tiles_kernel does.
// A grid smaller than the units is persistent (see kLogChunk).  Either way
// a pair's results are bitwise equal to a single-pair launch with the same
// geometry and unroll (ksplit 1).
struct BatchDesc {
    PairArgs a;
    int64_t unit_begin;
};
static_assert(sizeof(BatchDesc) <= IQA_BATCH_DESC_BYTES, "batch descriptor size");

constexpr int kBatchWaves = 4;   // waves per workgroup

// A pair whose waves split its tile groups' rows (rows_wave < NT).
__host__ __device__ __forceinline__ bool batch_coop(const PairArgs &a) { return a.rows_wave != a.NT; }

// A pair whose tile rows are longer than a tile's lanes.
__host__ __device__ __forceinline__ bool batch_wrap(const PairArgs &a) {
    return a.cols > 1 << a.log_grp;
}

// Work units of one pair.
__host__ __device__ __forceinline__ int64_t batch_units(const PairArgs &a) {
    const int64_t groups = (int64_t)a.ns * a.ngx;
    return batch_coop(a) ? groups : (groups + kBatchWaves - 1) / kBatchWaves;
}

// How units are dealt to the XCDs: chunks of 2^kLogChunk consecutive units go
// to the eight of them in turn, so that each gets its share of every pair, what
// is left after the last whole round is divided evenly, and an XCD's workgroups
// take its units in turn.  (One contiguous range of workgroups per XCD, as in
// the tile kernel, gave the second round of units to one XCD: 30 ragged pairs,
// 1.2 GB, 245 us against 177; units of unequal cost 203 against 180; the rest
// dealt as chunks: 22 ragged pairs 139 against 132.)  Chunks keep neighbouring
// tile groups, which share lines and DRAM pages, on one XCD: 128 units, or
// all of an XCD's where there are fewer (one 4096^2/128 pair, 1024 units: 24.2
// us, with chunks of 64 26.8, 32 27.1, 8 30.1, 1 33.5; four: 86.5, 64 90.0, 16
// 91.6; 512 pairs of 256^2/32, which share nothing: 45.6, 32 43.9).
constexpr int kLogChunk = 7;

template <int U, bool ODD = false>
__device__ __forceinline__ void batch_body(const BatchDesc *descs, int count, int64_t units) {
    __shared__ float4 lds[kBatchWaves][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // Fewer workgroups than XCDs are dealt to as if there were one.
    const int log_xcds = gridDim.x < kXcds ? 0 : kLogXcds;
    const uint32_t xcds = 1u << log_xcds, xcd = blockIdx.x & (xcds - 1);
    const uint32_t stride = (gridDim.x - xcd + xcds - 1) >> log_xcds;
    // The XCD's units: `whole` in chunks, then its share of what is left over.
    const int64_t whole = units >> (kLogChunk + log_xcds) << kLogChunk;
    const int64_t share = (units - (whole << log_xcds) + xcds - 1) >> log_xcds;
    for (int64_t i = blockIdx.x >> log_xcds; i < whole + share; i += stride) {
        const int64_t u = i < whole ? ((((i >> kLogChunk) << log_xcds) + xcd) << kLogChunk) +
                                          (i & ((1 << kLogChunk) - 1))
                                    : (whole << log_xcds) + xcd * share + (i - whole);
        if (u >= units) break;
        // Binary search for the pair whose units contain u (same in every wave).
        int lo = 0, hi = count - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (descs[mid].unit_begin <= u) lo = mid; else hi = mid - 1;
        }
        const int pi = __builtin_amdgcn_readfirstlane(lo);
        const PairArgs a = descs[pi].a;
        // A unit outside the pair's units (a unit count or pair count that
        // does not match the table) is skipped, never read.
        const int64_t g64 = u - descs[pi].unit_begin;
        if (g64 < 0 || g64 >= (ODD ? (int64_t)a.ns * a.ngx : batch_units(a))) continue;
        const bool leader = (lane & ((1 << a.log_grp) - 1)) == 0;
        if (!ODD && !batch_coop(a)) {
            const int64_t grp64 = g64 * kBatchWaves + wave;
            if (grp64 >= (int64_t)a.ns * a.ngx) continue;
            const int grp = (int)grp64;
            const int ty = udiv(grp, a.ngx_m, a.ngx);
            const int txg = grp - ty * a.ngx;
            const Sum4 s = batch_wrap(a) ? slice_sums<4, false, U, kBoth, true>(a, ty, txg, 0, lane)
                                     : slice_sums<4, false, U, kBoth, false>(a, ty, txg, 0, lane);
            const int tx = txg * tiles_per_wave(a) + (lane >> a.log_grp);
            if (leader && tx < a.ns)
                finalize<kBoth>(a, (int64_t)ty * a.ns + tx, s);
        } else {
            // Workgroup-uniform branch: every wave reaches both barriers.
            const int grp = (int)g64;
            const int ty = udiv(grp, a.ngx_m, a.ngx);
            const int txg = grp - ty * a.ngx;
            const Sum4 s = batch_wrap(a) ? slice_sums<4, ODD, U, kBoth, true>(a, ty, txg, wave, lane)
                                     : slice_sums<4, ODD, U, kBoth, false>(a, ty, txg, wave, lane);
            if (leader) lds[wave][lane >> a.log_grp] = float4{s.A, s.P, s.X, s.Y};
            __syncthreads();
            // Two waves finish the tiles at once, as in the tile kernel.
            if (wave < 2)
                finish_group<ODD>(a, lds, ty, txg, lane, [&](int64_t t, const Sum4 &r) {
                    if (wave == 0) {
                        finalize_lisi(a, t, r);
                        store_sums(a, t, r);
                    } else {
                        finalize_aug(a, t, r);
                    }
                });
            __syncthreads();   // the LDS slots are reused by the next unit
        }
    }
}

// The descriptor table in device memory (any number of pairs).  Bound by HBM: 30
// ragged pairs (1.2 GB) and 256 (10.8 GB) run at 6.7 TB/s, a plain read at 6.9.  Three
// waves per SIMD: more waves with fewer loads each in flight are slower on mixed
// batches (loads in batches of four, five waves: 223 us for the 30, 184 with eight).
template <int U>
__global__ __launch_bounds__(kBatchWaves * kWave, 3) void batch_kernel(const BatchDesc *descs,
                                                                       int count, int64_t units) {
    // No kernel writes the table while one reads it: constant memory, so that
    // a unit's descriptor is read into scalar registers.
    batch_body<U>((const BatchDesc *)(const IQA_CONSTANT BatchDesc *)(uintptr_t)descs, count, units);
}

// The pairs whose quads lie at any address (N_T % 4 != 0, images off 16 bytes):
// a unit is one of the tile kernel's workgroups, four waves on the quarters of a
// group's rows, so the results are bitwise a single launch's.  Launched one by
// one, small odd pairs are bound by their launches: 21 pairs of 240^2 to 2140^2,
// 9 of them odd, 0.22 GB (32 us of reads), took 69 us a run and take 48.
constexpr int kOddUnroll = 4;
static_assert(kAnyWaves == kBatchWaves, "an odd unit is a workgroup of the tile kernel");

__global__ __launch_bounds__(kBatchWaves * kWave) void odd_batch_kernel(const BatchDesc *descs,
                                                                        int count, int64_t units) {
    batch_body<kOddUnroll, true>(
        (const BatchDesc *)(const IQA_CONSTANT BatchDesc *)(uintptr_t)descs, count, units);
}

// Up to CAP descriptors passed by value in the kernel arguments: no table to
// copy to the device before the launch.  The waves read the descriptors
// straight from the kernel-argument segment.  Instantiated for CAP = 1, 4,
// IQA_BATCH_INLINE_MAX and kArgsMax: a launch uses the smallest that holds its batch,
// because the host-side cost of a launch grows with its argument size.
template <int CAP>
struct InlineDescs {
    BatchDesc d[CAP];
    int64_t units;
    int32_t count;
};

template <int U, int CAP>
__global__ __launch_bounds__(kBatchWaves * kWave) void batch_kernel_inline(InlineDescs<CAP> in) {
    batch_body<U>(in.d, in.count, in.units);
}

// ---------------------------------------------------------------------------
// Hierarchical aggregation (Eq. 3, Eq. 4)
// ---------------------------------------------------------------------------
//
// Eq. 3 and Eq. 4 recover the value of a larger tile (or of the whole image)
// from its child tiles.  Both weight each child's index by its own
// denominator, which is the same as adding the children's sums A, P, Sx, Sy
// and applying Eq. 1 / Eq. 2 to the totals; that is what these kernels do, from
// the sums iqa_tiles exports.
struct MergeArgs {
    const float *sums_in;   // ns*ns children, 4 floats each
    int64_t ns;             // children per side
    int64_t f;              // children per parent side
    float D, C2, C;
    float *lisi;
    float *aug;
    float *sums;
    int32_t parts;          // workgroups per parent
    float *ws;              // parts > 1: their partial sums and the parents' counters
};

__device__ __forceinline__ void finalize_merge(float D, float C2, float C, float *lisi, float *aug,
                                               float *sums, int64_t t, const Sum4 &s) {
    PairArgs k{};
    k.D = D;
    k.C2 = C2;
    k.C = C;
    k.lisi = lisi;
    k.aug = aug;
    k.sums = sums;
    finalize<kBoth>(k, t, s);
}

// f from 3 to 16: 2^log_g lanes per parent and LOADS children each, so a wave
// merges 64 >> log_g parents: one child per lane to f = 8, then a wave with four.
// (A workgroup per parent took 4.4 us for 48^2 parents of 4^2 children, where
// this is launch-bound; and 4.9 us for 32^2 of 16^2, 4.1 here.)
constexpr int kMergeThreads = 256;

template <int LOADS>
__global__ __launch_bounds__(kMergeThreads) void merge_small_kernel(MergeArgs m, int log_g) {
    const int np = (int)(m.ns / m.f), f = (int)m.f;
    const int lane = threadIdx.x & (kWave - 1);
    const int q = lane & ((1 << log_g) - 1);
    const int p = (int)(((int64_t)blockIdx.x * kMergeThreads + threadIdx.x) >> log_g);
    if (p >= np * np) return;   // the whole group
    const int py = p / np, px = p - py * np;
    const float4 *in =
        reinterpret_cast<const float4 *>(m.sums_in) + ((int64_t)py * m.ns + px) * f;
    float4 v[LOADS];
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
        const int c = q + u * kWave, cy = c / f, cx = c - cy * f;
        v[u] = c < f * f ? in[cy * m.ns + cx] : float4{0.f, 0.f, 0.f, 0.f};
    }
    const float4 w = wave_tree<LOADS>(v);
    const Sum4 s = group_allreduce<kBoth>(Sum4{w.x, w.y, w.z, w.w}, log_g);
    if (q == 0)
        finalize_merge(m.D, m.C2, m.C, m.lisi, m.aug, m.sums, p, s);
}

// f above 16.  A parent's children are cut into `parts` runs of
// part_children(), each added by kMergeThreads threads: a thread Kahan-adds
// every kMergeThreads-th child of the run, with eight loads in flight, the lanes
// and the four waves then add in a fixed order.  The runs' sums are added as a
// split tile's parts are (parts_sum).  (One run of any length took 393 us for the whole of a 512^2
// level, 4 MiB on one CU with one load in flight per thread.)
__host__ __device__ __forceinline__ int64_t part_children(int64_t f, int64_t parts) {
    return ((f * f + parts - 1) / parts + kMergeThreads - 1) / kMergeThreads * kMergeThreads;
}

// Thread t's share of run `part` of parent p, summed over its wave.
__device__ __forceinline__ float4 merge_run(const MergeArgs &m, int64_t p, int part, int t) {
    const int64_t np = m.ns / m.f;
    const int64_t py = p / np, px = p - py * np;
    const int64_t run = part_children(m.f, m.parts);
    const int64_t end = (part + 1) * run < m.f * m.f ? (part + 1) * run : m.f * m.f;
    const float4 *in =
        reinterpret_cast<const float4 *>(m.sums_in) + (py * m.ns + px) * m.f;
    int64_t c = part * run + t;
    int64_t cy = c / m.f, cx = c - cy * m.f;
    const int64_t dy = kMergeThreads / m.f, dx = kMergeThreads - dy * m.f;
    Acc acc = acc_zero();
    constexpr int kLoads = 8;
    for (int64_t left = run; left > 0; left -= kLoads * kMergeThreads) {
        float4 v[kLoads];
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            if (u * kMergeThreads >= left) break;   // the same for every thread
            v[u] = c < end ? in[cy * m.ns + cx] : float4{0.f, 0.f, 0.f, 0.f};
            c += kMergeThreads;
            cx += dx;
            cy += dy;
            if (cx >= m.f) {
                cx -= m.f;
                ++cy;
            }
        }
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            if (u * kMergeThreads >= left) break;
            cadd(acc.A, v[u].x);
            cadd(acc.P, v[u].y);
            cadd(acc.X, v[u].z);
            cadd(acc.Y, v[u].w);
        }
    }
    const Sum4 s = group_allreduce<kBoth>(fold(acc), 6);
    return float4{s.A, s.P, s.X, s.Y};
}

// The runs' sums of one parent, added by one wave.
template <typename Run>
__device__ __forceinline__ void merge_runs(const MergeArgs &m, int64_t p, int lane, Run run) {
    const Sum4 s = parts_sum<kBoth>(m.parts, 6, lane, run);
    if (lane == 0) finalize_merge(m.D, m.C2, m.C, m.lisi, m.aug, m.sums, p, s);
}

// One workgroup per run; the last of a parent's to finish adds them (the ticket
// of split_finish, one counter and one line per run and parent).
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(MergeArgs m) {
    __shared__ float4 waves[kMergeThreads / kWave];
    const int64_t p = blockIdx.x / m.parts;
    const int part = (int)(blockIdx.x - p * m.parts);
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const float4 v = merge_run(m, p, part, threadIdx.x);
    if (lane == 0) waves[wave] = v;
    __syncthreads();
    if (wave != 0) return;
    float4 w[4] = {waves[0], waves[1], waves[2], waves[3]};
    const float4 t = wave_tree<4>(w);
    if (m.parts == 1) {
        if (lane == 0)
            finalize_merge(m.D, m.C2, m.C, m.lisi, m.aug, m.sums, p, Sum4{t.x, t.y, t.z, t.w});
        return;
    }
    float4 *slots = reinterpret_cast<float4 *>(m.ws) + p * m.parts * (kLine / 16);
    if (lane == 0) store_coherent(slots + part * (kLine / 16), t);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(m.ws) - (kLine / 4) * (p + 1);
    wait_vmem();
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    uint32_t ticket = 0;
    if (lane == 0)
        ticket = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ticket = __builtin_amdgcn_readfirstlane(ticket);
    if (ticket != (uint32_t)(m.parts - 1)) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    merge_runs(m, p, lane, [&](int i) { return load_coherent(slots + i * (kLine / 16)); });
    if (lane == 0) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// All runs of a parent in one workgroup, four at a time, where there is no
// workspace (under capture); the same bits.
constexpr int kMergeLocalThreads = 4 * kMergeThreads;

__global__ __launch_bounds__(kMergeLocalThreads) void merge_local_kernel(MergeArgs m) {
    extern __shared__ float4 waves[];   // [parts][4]
    const int lane = threadIdx.x & (kWave - 1);
    const int team = threadIdx.x / kMergeThreads, t = threadIdx.x % kMergeThreads;
    for (int part = team; part < m.parts; part += kMergeLocalThreads / kMergeThreads) {
        const float4 v = merge_run(m, blockIdx.x, part, t);
        if (lane == 0) waves[part * 4 + t / kWave] = v;
    }
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    merge_runs(m, blockIdx.x, lane, [&](int i) {
        float4 w[4] = {waves[i * 4], waves[i * 4 + 1], waves[i * 4 + 2], waves[i * 4 + 3]};
        return wave_tree<4>(w);
    });
}

// A pyramid's next levels (f = 2 each) from one level's sums: a workgroup takes
// a block of 64 x 64 tiles and merges it up to six times, the levels' sums
// passing through LDS, so a level is read once and written once and a whole
// pyramid is one or two launches.  A parent is ((c00 + c01) + (c10 + c11)), as
// merge_small_kernel's lanes add four children.  (Seven levels over 192^2 tiles
// as merges of their own took 29 us on the GPU and 12 us of host time each.)
constexpr int kPyramidLevels = 6;
constexpr int kPyramidThreads = 1024;   // one per parent of the first level

struct PyramidArgs {
    const float *sums_in;   // ns*ns tiles, 4 floats each
    int32_t ns;             // tiles per side, a multiple of 2^levels
    int32_t levels;         // 1..kPyramidLevels
    int32_t nbx;            // blocks per side: ceil(ns / 64)
    float D, C2, C;
    float *lisi[kPyramidLevels];
    float *aug[kPyramidLevels];
    float *sums[kPyramidLevels];
};

__global__ __launch_bounds__(kPyramidThreads) void pyramid_kernel(PyramidArgs a) {
    __shared__ float4 level[kPyramidThreads];
    const int by = blockIdx.x / a.nbx, bx = blockIdx.x - by * a.nbx;
    int side = 32, n = a.ns / 2;   // parents per side: of the block, of the level
    int ty = threadIdx.x >> 5, tx = threadIdx.x & 31;
    auto add = [](const float4 &p, const float4 &q) {
        return float4{p.x + q.x, p.y + q.y, p.z + q.z, p.w + q.w};
    };
    for (int l = 0; l < a.levels; ++l) {
        const int py = by * side + ty, px = bx * side + tx;
        const bool mine = (int)threadIdx.x < side * side && py < n && px < n;
        float4 v{0.f, 0.f, 0.f, 0.f};
        if (mine) {
            if (l == 0) {
                const float4 *c = reinterpret_cast<const float4 *>(a.sums_in) +
                                  (int64_t)(2 * py) * a.ns + 2 * px;
                v = add(add(c[0], c[1]), add(c[a.ns], c[a.ns + 1]));
            } else {
                const float4 *c = level + (2 * ty) * (2 * side) + 2 * tx;
                v = add(add(c[0], c[1]), add(c[2 * side], c[2 * side + 1]));
            }
            finalize_merge(a.D, a.C2, a.C, a.lisi[l], a.aug[l], a.sums[l], (int64_t)py * n + px,
                           Sum4{v.x, v.y, v.z, v.w});
        }
        if (l + 1 == a.levels) break;   // the same for every thread
        __syncthreads();                // the level below has been read
        if ((int)threadIdx.x < side * side) level[threadIdx.x] = v;
        __syncthreads();
        side /= 2;
        n /= 2;
        ty = threadIdx.x / side;
        tx = threadIdx.x % side;
    }
}

// ---------------------------------------------------------------------------
// Streaming-read reference: the attainable HBM read rate on this GPU
// ---------------------------------------------------------------------------
//
// Each workgroup sums a contiguous chunk of float4s (several loads in flight
// per lane) and writes one float; the result is only there so that the loads
// cannot be removed.  Used to express the tile kernel's bandwidth as a
// fraction of what a plain read achieves.
__global__ __launch_bounds__(256) void read_ceiling_kernel(const float4 *__restrict__ src,
                                                           int64_t n4, int64_t per_block,
                                                           float *out) {
    const int64_t b0 = (int64_t)blockIdx.x * per_block;
    const int64_t b1 = b0 + per_block < n4 ? b0 + per_block : n4;
    float acc = 0.f;
    int64_t i = b0 + threadIdx.x;
    const IQA_GLOBAL char *f = global_bytes(reinterpret_cast<const float *>(src));
    for (; i + 3 * 256 < b1; i += 4 * 256) {
        const float4 a = vload<4>(f + 16 * i), b = vload<4>(f + 16 * (i + 256));
        const float4 c = vload<4>(f + 16 * (i + 512)), d = vload<4>(f + 16 * (i + 768));
        acc += (a.x + a.y + a.z + a.w) + (b.x + b.y + b.z + b.w) +
               (c.x + c.y + c.z + c.w) + (d.x + d.y + d.z + d.w);
    }
    for (; i < b1; i += 256) {
        const float4 a = vload<4>(f + 16 * i);
        acc += a.x + a.y + a.z + a.w;
    }
    for (int st = 32; st > 0; st >>= 1) acc += __shfl_xor(acc, st, kWave);
    __shared__ float part[4];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) out[blockIdx.x] = (part[0] + part[1]) + (part[2] + part[3]);
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

thread_local int g_last_hip_error = 0;

// Every launch goes through hipLaunchKernel and reports its own status (not a
// sticky error some earlier, unrelated call left behind).  The arguments take
// the kernel's own parameter types, so a mismatch does not compile.
template <typename T>
struct same_type {
    using type = T;
};

template <typename... P>
hipError_t launch_with_lds(void (*fn)(P...), unsigned grid, unsigned block, size_t lds,
                           hipStream_t s, typename same_type<P>::type... args) {
    void *argv[] = {static_cast<void *>(&args)...};
    return hipLaunchKernel(reinterpret_cast<const void *>(fn), dim3(grid), dim3(block), argv, lds,
                           s);
}

template <typename... P>
hipError_t launch_kernel(void (*fn)(P...), unsigned grid, unsigned block, hipStream_t s,
                         typename same_type<P>::type... args) {
    return launch_with_lds(fn, grid, block, 0, s, args...);
}

iqa_status hip_status(hipError_t e) {
    if (e == hipSuccess) return IQA_OK;
    g_last_hip_error = (int)e;
    return IQA_ERR_HIP;
}

using LaunchFn = hipError_t (*)(const KArgs &, uint64_t *, unsigned, hipStream_t);

template <int VEC, bool ANY, int WAVES, int U, int MODE, bool WRAP, bool SPLIT>
hipError_t launch_impl(const KArgs &a, uint64_t *, unsigned grid, hipStream_t s) {
    return launch_kernel(&tiles_kernel<VEC, ANY, WAVES, U, MODE, WRAP, SPLIT>, grid,
                         WAVES * kWave, s, a);
}

template <int VEC, int WAVES, int U, bool WRAP, bool SPLIT>
hipError_t launch_tl(const KArgs &a, uint64_t *tl, unsigned grid, hipStream_t s) {
    return launch_kernel(&tiles_kernel_tl<VEC, WAVES, U, WRAP, SPLIT>, grid, WAVES * kWave, s, a,
                         tl);
}

// What a launch needs, mapped onto the instantiated kernels.
struct Want {
    int mode;
    bool any;   // quads at any float address (Geometry::any)
    bool wrap, split, tl;
};

template <int VEC, bool ANY, int WAVES, int U, bool WRAP, bool SPLIT>
LaunchFn pick_mode(const Want &w) {
    if (w.tl) {
        if constexpr (VEC == 4 && !ANY) return &launch_tl<VEC, WAVES, U, WRAP, SPLIT>;
        return nullptr;
    }
    switch (w.mode) {
        case kLisi: return &launch_impl<VEC, ANY, WAVES, U, kLisi, WRAP, SPLIT>;
        case kAug: return &launch_impl<VEC, ANY, WAVES, U, kAug, WRAP, SPLIT>;
        default: return &launch_impl<VEC, ANY, WAVES, U, kBoth, WRAP, SPLIT>;
    }
}

template <int VEC, bool ANY, int WAVES, int U>
LaunchFn pick_shape(const Want &w) {
    if constexpr (VEC == 2) {   // 2 x 2 tiles only: one column
        if (w.wrap) return nullptr;
    } else if (w.wrap) {
        return w.split ? pick_mode<VEC, ANY, WAVES, U, true, true>(w)
                       : pick_mode<VEC, ANY, WAVES, U, true, false>(w);
    }
    return w.split ? pick_mode<VEC, ANY, WAVES, U, false, true>(w)
                   : pick_mode<VEC, ANY, WAVES, U, false, false>(w);
}

template <int VEC, bool ANY, int WAVES>
LaunchFn pick_unroll(int unroll, const Want &w) {
    switch (unroll) {
        case 4: return pick_shape<VEC, ANY, WAVES, 4>(w);
        case 8: return pick_shape<VEC, ANY, WAVES, 8>(w);
        default: return nullptr;
    }
}

// The instantiated launch shapes: waves 1/2/4/8 with unroll 4/8 and waves 16
// with unroll 4 for vec 4; for vec 2 and vec 1 with unroll 4 the any-address quad
// kernel for NT >= 4, four waves per workgroup whether one or four are asked for
// (an odd NT could only ask for one), and one wave of narrow loads below that.
// Each with and without a row split across workgroups.
// Timeline launches exist for the vec 4 shapes, fused mode.
LaunchFn pick(const iqa_launch_cfg &c, const Want &w) {
    if (c.vec == 4) {
        switch (c.waves) {
            case 1: return pick_unroll<4, false, 1>(c.unroll, w);
            case 2: return pick_unroll<4, false, 2>(c.unroll, w);
            case 4: return pick_unroll<4, false, 4>(c.unroll, w);
            case 8: return pick_unroll<4, false, 8>(c.unroll, w);
            case 16: return c.unroll == 4 ? pick_shape<4, false, 16, 4>(w) : nullptr;
            default: return nullptr;
        }
    }
    if (w.tl || c.unroll != 4 || !(c.waves == 1 || c.waves == 4)) return nullptr;
    if (w.any) return pick_shape<4, true, kAnyWaves, 4>(w);
    if (c.waves != 1) return nullptr;
    return c.vec == 2 ? pick_shape<2, false, 1, 4>(w) : pick_shape<1, false, 1, 4>(w);
}

bool is_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }
int ilog2(int64_t v) {
    int r = 0;
    while ((int64_t(1) << r) < v) ++r;
    return r;
}
int64_t next_pow2(int64_t v) { return int64_t(1) << ilog2(v); }

// Multiplier m = floor(2^(31 + ceil(log2 d)) / d) + 1 for udiv (1 <= d < 2^31).
uint32_t div_magic(int64_t d) {
    const int l = ilog2(d);
    return (uint32_t)(((uint64_t)1 << (31 + l)) / (uint64_t)d + 1);
}

bool param_ok(float v) {
    return std::isfinite(v) && v > 0.f && std::fpclassify(v) == FP_NORMAL;
}

bool aligned(const void *p, size_t b) { return (reinterpret_cast<uintptr_t>(p) % b) == 0; }

iqa_status check_shape(int64_t N, int64_t NT) {
    if (N <= 0 || NT <= 0 || N > IQA_MAX_N || NT > N || N % NT != 0) return IQA_ERR_SHAPE;
    return IQA_OK;
}

struct Geometry {
    int64_t ns, ht, ngx, groups, grid;
    int log_grp;
    int cols;
    bool any, wrap;
};

iqa_status geometry(int64_t N, int64_t NT, const iqa_launch_cfg &c, Geometry &g) {
    if (!(c.vec == 1 || c.vec == 2 || c.vec == 4) || NT % c.vec) return IQA_ERR_CONFIG;
    if (!is_pow2(c.seg) || !is_pow2(c.rp) || (int64_t)c.seg * c.rp > kWave) return IQA_ERR_CONFIG;
    if (!is_pow2(c.waves) || c.waves > 16) return IQA_ERR_CONFIG;
    if (c.ksplit < 1 || NT % ((int64_t)c.waves * c.ksplit) != 0) return IQA_ERR_CONFIG;
    // vec 2 and vec 1 stand for images whose rows or tiles 16-byte loads do
    // not fit.  From NT = 4 on they run quads at any float address: the same
    // lanes per tile, one 16-byte load at 4-byte alignment in place of four
    // 4-byte or two 8-byte ones.
    g.any = c.vec < 4 && NT >= 4;
    if (pick(c, Want{kBoth, g.any, false, false, false}) == nullptr) return IQA_ERR_CONFIG;
    g.ns = N / NT;
    g.log_grp = ilog2((int64_t)c.seg * c.rp);
    g.ht = kWave >> g.log_grp;
    g.ngx = (g.ns + g.ht - 1) / g.ht;
    g.groups = g.ns * g.ngx;
    g.grid = g.groups * c.ksplit;
    g.cols = (int)(g.any ? (NT + 3) / 4 : NT / c.vec);
    g.wrap = g.cols > 1 << g.log_grp;
    if (g.grid > (int64_t)INT_MAX) return IQA_ERR_CONFIG;
    return IQA_OK;
}

// Built-in launch shape for (N, NT), for shapes the autotuner has not
// measured: the widest vector the images' alignment and NT allow (vec 2 and
// vec 1 run any-address quads), four waves per workgroup, and batches of four
// rows.  Two rules follow.
//
// Lanes per tile.  A wave covers as many adjacent tiles as fit, one row of
// quads each, unless that leaves less than a workgroup per CU or too many
// items per lane; then it takes fewer tiles and more rows of each.  The lines,
// in us: 256 workgroups (1000^2/100: 100 workgroups 5.7, 50 6.1; 3000^2/100:
// 450 workgroups 13.9, 900 14.5), and 8 items where a row is at most 16 quads
// (3840^2/40: 5 items 21.1, 10 items 21.9).  At 32 lanes a row, two rows if a
// tile row is whole 128-byte lines (3840^2/96: 21.0, one row of two tiles
// 23.3), else one row of two tiles, which share the line between them
// (3840^2/120: 20.6, two rows above 22).  Any-address quads: 6 items for rows
// of at most 8 quads (8190^2/30: 4 items 80.0, 8 items 84.0), and two rows at 32
// lanes (8190^2/90: 85.8 and 88.2).  Rows of 13 to 16 quads keep 16 lanes, up to
// 16 items, where that makes one workgroup per CU or 1.5 to 2 (16 lanes and 32: 256
// of them, 1600^2/50 6.1 and 6.3; 400, 2000^2/50 7.7 and 8.3; 462, 2394^2/57 9.5 and 10.2; 484, 2508^2/57 9.9 and
// 10.4, 2772^2/63 11.7 and 11.7; but 315, 2135^2/61 9.7 and 9.0; 564, 2350^2/50
// 10.2 and 9.8; 540, 2385^2/53 11.1 and 10.4, 2835^2/63 14.5 and 13.2; 1600,
// 4000^2/50 21.5 and 20.7); 9 to 12 quads do not (484, 1804^2/41 7.2 and 7.0,
// 1980^2/45 7.8 and 7.7; 540, 2025^2/45 9.4 and 8.4).
//
// Eight waves per workgroup instead of four, unsplit, where there is a workgroup
// for more than half of the CUs and at most one for each, from 16 items per lane
// (of four) to 64 (of eight).  (1920^2/160, 144 workgroups: 8.9 us, split four
// ways 10.7, unsplit 11.4; 2800^2/200, 196: 13.0, 14.4, 14.8; 3072^2/256, 144:
// 16.0, 17.7, 18.0; 3200^2/200, 256: 15.7, four waves 16.6; but 1920^2/120, 15
// items, 256: 8.0 and 7.8; 2880^2/160, 324: 16.3 and 14.9; 4800^2/400, 78 items
// of eight, 144: 36.2, split 33.4.)  For a few less, which would be split in only
// two, up to 24 items of eight (121 workgroups: 1760^2/160 8.6 and 9.1, 2112^2/192
// 10.2 and 10.6; 2200^2/200 11.3 and 11.2, 3520^2/320 22.1 and 20.0; 100 of them,
// split in five: 1600^2/160 8.5 and 8.1).  Tiles too small to be split, from
// 14 items per lane (of four), take sixteen waves on up to 200 workgroups
// (1152^2/128, 81: 5.7, four waves 6.4; 1792^2/128, 196: 6.9 and 7.5; 1120^2/112:
// 5.6 and 6.1; 2048^2/128, 256, eight waves 7.9, sixteen 8.1).
//
// Splits.  A tile whose waves would each make more than 24 items is split over
// workgroups if the launch has less than one of four waves per CU: into the fewest parts that give it that, as long as a lane keeps 3
// items.  (Unsplit against split: 1000^2/100, 13 items, 5.7 and 6.2;
// 3000^2/300, 88 items, 23.4 and 15.6.)  Counts from one workgroup per CU to
// nearly two are passed over: some CUs would have twice the work of others
// (6000^2/1500: 240 workgroups 49.6, 400 54.3, 1200 51.5).  A few deeply split
// tiles take eight waves per workgroup, so that fewer parts are added at the
// end (2048^2/2048: 128 parts of eight waves 11.6, 256 of four 12.6).
iqa_launch_cfg default_cfg(int64_t N, int64_t NT, const float *x, const float *y) {
    iqa_launch_cfg c{};
    c.vec = 1;
    if (NT % 2 == 0 && aligned(x, 8) && aligned(y, 8)) c.vec = 2;
    if (NT % 4 == 0 && aligned(x, 16) && aligned(y, 16)) c.vec = 4;
    c.unroll = 4;
    c.waves = NT % 4 == 0 ? 4 : 1;
    c.ksplit = 1;
    int64_t wg_waves = c.waves;
    const bool any = c.vec < 4 && NT >= 4;
    const int64_t cols = any ? (NT + 3) / 4 : NT / c.vec;
    const int64_t row_lanes = std::min<int64_t>(kWave, next_pow2(cols));
    const int64_t ns = N / NT;
    if (any) wg_waves = kAnyWaves;
    const int64_t rows = (NT + wg_waves - 1) / wg_waves;   // per wave
    int64_t lanes = row_lanes;
    auto workgroups = [&] { return ns * ((ns * lanes + kWave - 1) / kWave); };
    auto items = [&](int64_t r) {
        return (r * (cols > kWave ? cols : row_lanes) + lanes - 1) / lanes;
    };
    while (lanes < kWave) {
        const bool few = workgroups() * wg_waves < 1024;
        const bool rounds = workgroups() <= 256 || (workgroups() > 384 && workgroups() <= 512);
        const int64_t most = !any ? 8 : row_lanes <= 8 ? 6 : cols >= 13 && rounds ? 16 : 8;
        const bool long_lane = row_lanes <= 16 && items(rows) > most;
        const bool whole_lines = row_lanes == 32 && (any || NT % 32 == 0);
        if (!few && !long_lane && !whole_lines) break;
        lanes *= 2;
    }
    c.seg = (int)std::min<int64_t>(lanes, next_pow2(NT / c.vec));
    c.rp = (int)(lanes / c.seg);
    // HIP launches fewer than 2^32 work items (131072^2/4: one wave).
    if (c.vec == 4 && workgroups() * wg_waves * kWave > (int64_t)UINT32_MAX) {
        c.waves = 1;
        return c;
    }
    const int64_t tiles = ns * ns;
    if (c.vec == 4 && lanes == kWave && workgroups() <= 256) {
        const int64_t wgs = workgroups(), each = items(rows);
        if (NT % 16 == 0 && each >= 14 && each <= 24 && wgs <= 200) c.waves = 16;
        else if (NT % 8 == 0 && each >= 16 && wgs > 112 && items(NT / 8) <= (wgs > 128 ? 64 : 24))
            c.waves = 8;
        if (c.waves > 4) return c;
    }
    if (workgroups() * wg_waves >= 1024 || items(rows) <= 24 || lanes < kWave) return c;
    if (c.vec == 4 && tiles <= 16 && NT % 8 == 0) c.waves = 8, wg_waves = 8;
    auto enough = [&](int64_t wgs) { return wgs >= 225 && (wgs <= 256 || wgs >= 448); };
    // Parts are equal: divisors of a wave's (any: a workgroup's) rows.  At most 4096 slices of a tile
    // (see launch_local) and as many parts in all as the fixed scratch holds.
    constexpr int64_t kMostParts = (IQA_NOALLOC_SCRATCH_BYTES - (64 << 10)) / 16;
    const int32_t per = (int32_t)(NT / c.waves);
    for (int32_t ks = 1; ks <= per && ks * wg_waves <= 4096 && tiles * ks <= kMostParts; ++ks) {
        if (per % ks != 0) continue;
        if (items((NT / ks + wg_waves - 1) / wg_waves) < 3) break;
        c.ksplit = ks;
        if (enough(tiles * ks)) break;
    }
    return c;
}

// Whether the stream's workspace belongs to (N, NT)'s default launch whatever
// the stream is doing: the shapes documented to need iqa_prepare before a
// capture, those that powers of two split.  Other default splits use a
// workspace of their own, and none under capture (see Ws).
bool split_needs_prepare(int64_t N, int64_t NT, int64_t vec) {
    const int64_t seg = std::min<int64_t>(kWave, next_pow2(NT / vec));
    const int64_t rp = std::min<int64_t>(2, kWave / seg);
    const int64_t ht = kWave / seg / rp;
    const int64_t ns = N / NT;
    int64_t kw = 1;
    while (kw < (vec == 4 ? 16 : 4) && NT % (kw * 2) == 0 && NT / (rp * kw * 2) >= 16) kw *= 2;
    if (vec != 4 && kw > 1) kw = NT % 4 == 0 ? 4 : 1;
    return ns * ((ns + ht - 1) / ht) * kw < 1024 && NT % (kw * 2) == 0 && NT / (rp * kw * 2) >= 4;
}

// Tuned launch shapes.  The autotuner's measurements on gfx950 are compiled in
// (tuned_table.inc, generated by the build from the tuner's JSON cache);
// entries registered at run time take precedence.  kind 0 = single-pair
// launches, kind 1 = per-pair geometry in batches; N == 0 matches any N.
struct TunedEntry {
    int64_t N, NT;
    int kind;
    iqa_launch_cfg cfg;
};
#if __has_include("tuned_table.inc")
#include "tuned_table.inc"
#else
static const TunedEntry kTuned[] = {{-1, -1, -1, {0, 0, 0, 0, 0, 0}}};
static const int kTunedCount = 0;
static const int64_t kTunedBatchWaves = 0;
#endif

std::mutex g_tune_mutex;
std::map<std::tuple<int64_t, int64_t, int>, iqa_launch_cfg> g_tuned;

// The per-pair geometries the batch kernel can run: vec 4, no row split,
// unroll 8, and one wave per tile group or the workgroup's four waves on each.
constexpr int kBatchUnroll = 8;

bool batch_geometry_ok(const iqa_launch_cfg &c) {
    return c.vec == 4 && c.ksplit == 1 && c.unroll == kBatchUnroll &&
           (c.waves == 1 || c.waves == kBatchWaves);
}

bool tuned_lookup(int64_t N, int64_t NT, int kind, iqa_launch_cfg *out) {
    {
        std::lock_guard<std::mutex> lock(g_tune_mutex);
        for (int64_t n : {N, int64_t(0)}) {
            auto it = g_tuned.find(std::make_tuple(n, NT, kind));
            if (it != g_tuned.end()) {
                *out = it->second;
                return true;
            }
        }
    }
    for (int64_t n : {N, int64_t(0)}) {
        for (int i = 0; i < kTunedCount; ++i) {
            const TunedEntry &e = kTuned[i];
            if (e.N == n && e.NT == NT && e.kind == kind) {
                Geometry g{};
                if (geometry(N, NT, e.cfg, g) != IQA_OK) continue;
                if (kind != IQA_TUNE_SINGLE && !batch_geometry_ok(e.cfg)) continue;
                *out = e.cfg;
                return true;
            }
        }
    }
    return false;
}

// A split default launch with the contract of split launches: a tuned shape,
// or one that split_needs_prepare names.
bool tuned_or_prepared(int64_t N, int64_t NT, const iqa_launch_cfg &c, const float *x,
                       const float *y) {
    iqa_launch_cfg t;
    if (aligned(x, 16) && aligned(y, 16) && tuned_lookup(N, NT, IQA_TUNE_SINGLE, &t)) return true;
    return split_needs_prepare(N, NT, c.vec);
}

iqa_launch_cfg pick_cfg(int64_t N, int64_t NT, const float *x, const float *y) {
    iqa_launch_cfg c;
    if (aligned(x, 16) && aligned(y, 16) && tuned_lookup(N, NT, 0, &c)) return c;
    return default_cfg(N, NT, x, y);
}

// Per-pair geometry inside a batch: units of about 128 KiB of input, so that a
// batch's units cost alike whatever its shapes: four tile groups of one wave
// each for small tiles, one group whose rows four waves share for larger ones.
iqa_launch_cfg batch_cfg(int64_t N, int64_t NT) {
    iqa_launch_cfg c;
    if (tuned_lookup(N, NT, 1, &c)) return c;
    c.vec = 4;
    c.waves = NT <= 40 ? 1 : kBatchWaves;
    c.unroll = kBatchUnroll;
    c.ksplit = 1;
    const int64_t lpt = NT / 4;
    c.seg = (int)std::min<int64_t>(kWave, next_pow2(lpt));
    const int64_t tpw = kWave / c.seg;
    const int64_t want = (int64_t(32) << 10) * c.waves / (8 * NT * NT);
    int64_t ht = 1;
    while (ht * 2 <= tpw && ht * 2 <= want && ht * 2 <= next_pow2(N / NT)) ht *= 2;
    c.rp = (int)(tpw / ht);
    return c;
}

// Per-pair geometry in the server's batches: its own tuned entries (chosen
// for a lone pair's latency), else the ragged-batch geometry.
iqa_launch_cfg serve_cfg(int64_t N, int64_t NT) {
    iqa_launch_cfg c;
    if (tuned_lookup(N, NT, IQA_TUNE_SERVE, &c)) return c;
    return batch_cfg(N, NT);
}

// Per (device, stream) workspace for split tiles: a counter region (ticket
// counters only) followed by a partial-sum region.  A launch uses its
// workspace from its first workgroup to its last, and launches on one stream
// run one after the other, so one buffer per stream is enough; concurrent
// streams get their own (hipStreamPerThread: one per host thread).  A new
// buffer is cleared on its stream before first use, and since each launch leaves its counters at zero, the counter region
// stays all zeros between launches whatever shapes share it.  A buffer that
// is outgrown is kept, not freed: a graph captured earlier may still launch
// kernels that use it.
struct Workspace {
    void *ptr = nullptr;
    size_t cnt_bytes = 0;    // counter region, at ptr
    size_t part_bytes = 0;   // partial-sum region, at ptr + cnt_bytes
    bool told = false;       // iqa_prepare was called on the stream with a configuration
};
std::mutex g_ws_mutex;
std::map<std::tuple<int, void *, int, bool>, Workspace> g_ws;
std::vector<void *> g_ws_retired;

// hipStreamPerThread is one handle for a stream of every host thread, so its
// buffers are a thread's too.  Threads that use it are numbered; a thread that
// ends waits for its streams and hands its number, and so its buffers, on.
std::mutex g_thread_mutex;
std::vector<bool> g_thread_used;   // by number, from 0

class ThreadNumber {
public:
    // Of this thread, which uses its stream of device `dev`.
    int on(int dev) {
        if (number_ < 0) {
            std::lock_guard<std::mutex> lock(g_thread_mutex);
            number_ = (int)(std::find(g_thread_used.begin(), g_thread_used.end(), false) -
                            g_thread_used.begin());
            if (number_ == (int)g_thread_used.size()) g_thread_used.push_back(false);
            g_thread_used[number_] = true;
        }
        if (std::find(devices_.begin(), devices_.end(), dev) == devices_.end())
            devices_.push_back(dev);
        return number_;
    }
    ~ThreadNumber() {
        if (number_ < 0) return;
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;   // leave others' captures alone
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        for (int dev : devices_) {
            // A stream that cannot be waited for keeps the number.
            if (hipSetDevice(dev) != hipSuccess ||
                hipStreamSynchronize(hipStreamPerThread) != hipSuccess)
                return;
        }
        std::lock_guard<std::mutex> lock(g_thread_mutex);
        g_thread_used[number_] = false;
    }

private:
    int number_ = -1;
    std::vector<int> devices_;
};
thread_local ThreadNumber t_thread;

// Split launches of at most this many workgroups (one round on gfx950's 256
// CUs at four workgroups each) add their parts by ticket, within the launch;
// larger ones store their partials and a combine launch adds them (see
// split_finish for why).
constexpr int64_t kTicketMaxGrid = 1024;

int split_mode(const Geometry &g, const iqa_launch_cfg &c) {
    if (c.ksplit <= 1) return kSplitNone;
    return g.grid <= kTicketMaxGrid ? kSplitTicket : kSplitCombine;
}

struct SplitNeed {
    size_t cnt_bytes = 0, part_bytes = 0;   // 0, 0: the launch does not split
};

SplitNeed split_need(const Geometry &g, const iqa_launch_cfg &c) {
    SplitNeed n;
    const int m = split_mode(g, c);
    if (m == kSplitNone) return n;
    if (m == kSplitTicket) n.cnt_bytes = (size_t)(g.groups * kLine);
    n.part_bytes = (size_t)(g.groups * c.ksplit * part_entries(m, g.ht)) * 4 * sizeof(float);
    return n;
}

size_t round_up(size_t v, size_t m) { return (v + m - 1) / m * m; }

// Whether s is being captured (or cannot say).
bool capturing(hipStream_t s) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (s == nullptr) return false;
    return hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone;
}

// Least sizes of a workspace's regions: what any launch with ticket counters
// needs, so that a buffer rarely grows.
constexpr size_t kCounterBytes = 64 << 10, kPartBytes = 128 << 10;

// The launches that can do without a workspace (run and merge) keep buffers for
// this many streams at most, of at most two sizes each; on further streams they
// do without.
constexpr int kMostOwn = 128;
int g_own_buffers = 0;

std::tuple<int, void *, int, bool> ws_key(int dev, hipStream_t s, bool own) {
    const int thread = s == hipStreamPerThread ? t_thread.on(dev) : -1;
    return std::make_tuple(dev, (void *)s, thread, own);
}

// *part receives the partial-sum region; the counter region ends where it
// starts.  `own`: a buffer of the launches that can do without.  The caller
// holds g_ws_mutex.
iqa_status workspace_for(hipStream_t s, bool own, const SplitNeed &need, float **part) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_status(e);
    const auto key = ws_key(dev, s, own);
    if (own && g_own_buffers >= kMostOwn) {
        const auto it = g_ws.find(key);
        if (it == g_ws.end() || !it->second.ptr) return IQA_ERR_SCRATCH;
    }
    Workspace &w = g_ws[key];
    if (w.cnt_bytes < need.cnt_bytes || w.part_bytes < need.part_bytes) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (s != nullptr) {
            e = hipStreamIsCapturing(s, &cs);
            if (e != hipSuccess) return hip_status(e);
        }
        if (cs != hipStreamCaptureStatusNone) return IQA_ERR_CAPTURE;
        const size_t cb = round_up(std::max({need.cnt_bytes, w.cnt_bytes, kCounterBytes}), 4096);
        size_t pb = round_up(std::max({need.part_bytes, w.part_bytes, kPartBytes}), 4096);
        if (own && pb > kPartBytes) pb = std::max(pb, (size_t)IQA_NOALLOC_SCRATCH_BYTES);
        void *p = nullptr;
        // A launch that needs no preparation may come while another stream is
        // being captured: the allocation must not disturb that.
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (own) (void)hipThreadExchangeStreamCaptureMode(&mode);
        e = hipMalloc(&p, cb + pb);
        if (own) (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (e != hipSuccess) return hip_status(e);
        e = hipMemsetAsync(p, 0, cb + pb, s);
        if (e != hipSuccess) {
            (void)hipFree(p);
            return hip_status(e);
        }
        if (w.ptr) g_ws_retired.push_back(w.ptr);
        else if (own) ++g_own_buffers;
        w.ptr = p;
        w.cnt_bytes = cb;
        w.part_bytes = pb;
    }
    *part = reinterpret_cast<float *>(static_cast<char *>(w.ptr) + w.cnt_bytes);
    return IQA_OK;
}

// Whether a launch that can do without has a workspace.  The caller holds
// g_ws_mutex.
bool own_workspace(hipStream_t s, const SplitNeed &need, float **part) {
    const int err = g_last_hip_error;
    if (workspace_for(s, true, need, part) == IQA_OK) return true;
    (void)hipGetLastError();
    g_last_hip_error = err;
    return false;
}

// Whether the caller of launches on s has called iqa_prepare there with a
// configuration, and so knows of the workspace that they share.
bool prepared_with_cfg(hipStream_t s) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    std::lock_guard<std::mutex> lock(g_ws_mutex);
    const auto it = g_ws.find(ws_key(dev, s, false));
    return it != g_ws.end() && it->second.told;
}

// Scratch of the no-allocation entry point: a fixed array in device memory,
// one copy per GPU, held until the process ends.  It starts zeroed (the
// loader clears the array), and every launch leaves its ticket counters at
// zero.  Its device address comes from hipGetSymbolAddress, once per device,
// with that device current; host code never uses the array's name otherwise.
static __device__ __align__(256) float scratch[IQA_NOALLOC_SCRATCH_BYTES / sizeof(float)];

// The first kScratchCounterBytes of the array are the counter region (the
// partial-sum region starts right after it), the rest holds partial sums.
constexpr size_t kScratchCounterBytes = 64 << 10;

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

// The caller holds g_scratch_mutex.
iqa_status scratch_for_current_device(float **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_status(e);
    if (dev < 0 || dev >= kMaxDevices) return IQA_ERR_CONFIG;
    if (g_scratch_ptr[dev] == nullptr) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_status(e);
        if (p == nullptr) return IQA_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = static_cast<float *>(g_scratch_ptr[dev]);
    return IQA_OK;
}

void fill_pair(PairArgs &a, const float *x, const float *y, int64_t N, int64_t NT, float D,
               float C1, float C2, float C, float *lisi, float *aug, float *sums,
               const iqa_launch_cfg &c, const Geometry &g) {
    a.x = x;
    a.y = y;
    a.lisi = lisi;
    a.aug = aug;
    a.sums = sums;
    a.D = D;
    a.C1 = C1;
    a.C2 = C2;
    a.C = C;
    a.N = (int32_t)N;
    a.NT = (int32_t)NT;
    a.ns = (int32_t)g.ns;
    a.ngx = (int32_t)g.ngx;
    a.ngx_m = div_magic(g.ngx);
    a.log_grp = g.log_grp;
    a.rows_wave = (int32_t)(NT / ((g.any ? 1 : (int64_t)c.waves) * c.ksplit));
    const int64_t lanes = int64_t(1) << g.log_grp;
    const int64_t pitch = g.wrap ? g.cols : next_pow2(g.cols);
    a.cols = g.cols;
    a.pitch = (int32_t)pitch;
    a.pitch_m = (uint32_t)(((int64_t(1) << 31) + pitch - 1) / pitch);
    if (!g.any) {
        const int64_t places = a.rows_wave * pitch;
        a.items = (places + lanes - 1) / lanes;
        const int64_t shift = a.items * lanes - places;
        a.lead_rows = (int32_t)((shift + pitch - 1) / pitch);
        a.lead = (int32_t)(a.lead_rows * pitch - shift);
    }
    const int64_t quad_bytes = 4 * (g.any ? 4 : c.vec);
    a.step = (int32_t)(g.wrap ? lanes * quad_bytes : lanes / pitch * N * 4);
}

hipError_t launch_combine(const KArgs &a, int mode, const Geometry &g, hipStream_t s) {
    void (*fn)(KArgs) = mode == kLisi  ? &combine_kernel<kLisi>
                        : mode == kAug ? &combine_kernel<kAug>
                                       : &combine_kernel<kBoth>;
    return launch_kernel(fn, (unsigned)g.groups, kWave, s, a);
}

// LDS of a tiles_local_kernel workgroup: 16 bytes per slice of its tile.
constexpr size_t kLocalLdsMax = 64 << 10;

int part_slices(const iqa_launch_cfg &c, const Geometry &g) { return g.any ? kAnyWaves : c.waves; }

size_t local_lds(const iqa_launch_cfg &c, const Geometry &g) {
    return (size_t)part_slices(c, g) * c.ksplit * sizeof(float4);
}

// Shapes whose default launch splits without split_needs_prepare: whether this
// configuration can run without a workspace too.
bool local_ok(const iqa_launch_cfg &c, const Geometry &g) {
    return g.ht == 1 && c.unroll == 4 && (c.vec == 4 || g.any) && local_lds(c, g) <= kLocalLdsMax &&
           (c.waves == 1 || c.waves == 4 || c.waves == 8);
}

template <bool ANY, bool WRAP>
hipError_t launch_local_mode(const KArgs &a, int mode, const iqa_launch_cfg &c, const Geometry &g,
                             hipStream_t s) {
    void (*fn)(KArgs, int) = mode == kLisi  ? &tiles_local_kernel<ANY, 4, kLisi, WRAP>
                             : mode == kAug ? &tiles_local_kernel<ANY, 4, kAug, WRAP>
                                            : &tiles_local_kernel<ANY, 4, kBoth, WRAP>;
    return launch_with_lds(fn, (unsigned)g.groups, kLocalWaves * kWave, local_lds(c, g), s, a,
                           part_slices(c, g));
}

hipError_t launch_local(const KArgs &a, int mode, const iqa_launch_cfg &c, const Geometry &g,
                        hipStream_t s) {
    if (g.any) {
        return g.wrap ? launch_local_mode<true, true>(a, mode, c, g, s)
                      : launch_local_mode<true, false>(a, mode, c, g, s);
    }
    return g.wrap ? launch_local_mode<false, true>(a, mode, c, g, s)
                  : launch_local_mode<false, false>(a, mode, c, g, s);
}

bool same_cfg(const iqa_launch_cfg &a, const iqa_launch_cfg &b) {
    return a.vec == b.vec && a.waves == b.waves && a.unroll == b.unroll && a.seg == b.seg &&
           a.rp == b.rp && a.ksplit == b.ksplit;
}

// Where a launch's split workspace comes from.
enum class Ws {
    kLibrary,   // the per-(device, stream) buffer, grown on demand
    kScratch,   // the fixed scratch array (no allocation; bounded size)
    kPrepare,   // only allocate the library buffer, launch nothing
};

// A default launch that splits without split_needs_prepare must not put the
// rules of split launches on its caller (prepare before a capture, no other
// split work beside a graph's replay or on the scratch array).  Run eagerly on
// a stream it has a buffer of its own there, which launches on that stream use
// one after the other and no graph ever holds; captured, or through the
// no-allocation entry point, it runs without a workspace (launch_local),
// bitwise the same.  So does the default configuration passed back, unless
// iqa_prepare was told of a configuration on that stream.
iqa_status run(const float *x, const float *y, int64_t N, int64_t NT, float D, float C1,
               float C2, float C, float *lisi, float *aug, float *sums,
               const iqa_launch_cfg *cfg_in, void *stream, Ws ws, uint64_t *tl = nullptr) {
    iqa_launch_cfg c = cfg_in ? *cfg_in : pick_cfg(N, NT, x, y);
    Geometry g{};
    iqa_status st = geometry(N, NT, c, g);
    if (st != IQA_OK) return st;
    if (ws != Ws::kPrepare) {
        if (!aligned(x, 4 * c.vec) || !aligned(y, 4 * c.vec)) return IQA_ERR_ALIGN;
    }
    int mode = ((lisi || sums) ? kLisi : 0) | ((aug || sums) ? kAug : 0);
    if (mode == 0) mode = kBoth;
    LaunchFn fn = pick(c, Want{mode, g.any, g.wrap, c.ksplit > 1, tl != nullptr});
    if (!fn) return IQA_ERR_CONFIG;
    hipStream_t s = static_cast<hipStream_t>(stream);

    KArgs a{};
    const SplitNeed need = split_need(g, c);
    bool own = false, local = false;
    if (c.ksplit > 1 && (!cfg_in || (!tl && same_cfg(c, pick_cfg(N, NT, x, y)))) &&
        local_ok(c, g) && !tuned_or_prepared(N, NT, c, x, y)) {
        own = true;
        local = ws == Ws::kScratch || (ws == Ws::kLibrary && capturing(s));
        if (cfg_in && (ws == Ws::kPrepare || (ws == Ws::kLibrary && local && prepared_with_cfg(s))))
            own = local = false;
    }
    // The workspace (or scratch) stays locked until the launches are
    // enqueued: a combine-mode split is two launches, and another host
    // thread's split launches on the same stream must not come between them.
    std::unique_lock<std::mutex> ws_lock(g_ws_mutex, std::defer_lock);
    std::unique_lock<std::mutex> scratch_lock(g_scratch_mutex, std::defer_lock);
    if (need.part_bytes > 0 && !local) {
        if (ws == Ws::kScratch) {
            if (need.cnt_bytes > kScratchCounterBytes ||
                need.part_bytes > IQA_NOALLOC_SCRATCH_BYTES - kScratchCounterBytes)
                return IQA_ERR_SCRATCH;
            scratch_lock.lock();
            float *base = nullptr;
            st = scratch_for_current_device(&base);
            if (st != IQA_OK) return st;
            a.ws = reinterpret_cast<float *>(reinterpret_cast<char *>(base) + kScratchCounterBytes);
        } else {
            ws_lock.lock();
            if (!own) {
                st = workspace_for(s, false, need, &a.ws);
                if (st != IQA_OK) return st;
            } else if (!own_workspace(s, need, &a.ws)) {
                ws_lock.unlock();
                local = true;
            }
        }
    }
    if (ws == Ws::kPrepare) {
        if (cfg_in && ws_lock.owns_lock()) {
            int dev = 0;
            if (hipGetDevice(&dev) == hipSuccess) g_ws[ws_key(dev, s, false)].told = true;
        }
        return IQA_OK;
    }

    fill_pair(a, x, y, N, NT, D, C1, C2, C, lisi, aug, sums, c, g);
    a.smode = split_mode(g, c);
    a.ks = c.ksplit;
    a.ks_m = div_magic(c.ksplit);
    if (local) return hip_status(launch_local(a, mode, c, g, s));
    hipError_t e = fn(a, tl, (unsigned)g.grid, s);
    if (e == hipSuccess && a.smode == kSplitCombine) e = launch_combine(a, mode, g, s);
    return hip_status(e);
}

// One level of merging.  Which kernel, and in how many runs, is a function of
// (ns, f) alone.  f == 2 is a pyramid of one level: one thread per parent (a
// workgroup each took 42 us for 256^2 parents).  Runs of 4096 children, as long
// as the launch has fewer than 1024 workgroups: 16 loads per thread, below which
// the ticket costs more than it saves.
constexpr int64_t kRunChildren = 4096, kMergeMaxGrid = 1024;

iqa_status merge(const float *sums_in, int64_t ns, int64_t f, float D, float C2, float C,
                 float *lisi, float *aug, float *sums, hipStream_t s) {
    const int64_t parents = (ns / f) * (ns / f);
    if (f == 2) {
        PyramidArgs a{};
        a.sums_in = sums_in;
        a.ns = (int32_t)ns;
        a.levels = 1;
        a.nbx = (int32_t)((ns + 63) / 64);
        a.D = D;
        a.C2 = C2;
        a.C = C;
        a.lisi[0] = lisi;
        a.aug[0] = aug;
        a.sums[0] = sums;
        return hip_status(
            launch_kernel(&pyramid_kernel, (unsigned)(a.nbx * a.nbx), kPyramidThreads, s, a));
    }
    MergeArgs m{sums_in, ns, f, D, C2, C, lisi, aug, sums, 1, nullptr};
    if (f <= 16) {
        const int log_g = std::min(ilog2(f * f), 6);
        const int64_t per = kMergeThreads >> log_g;
        return hip_status(launch_kernel(f <= 8 ? &merge_small_kernel<1> : &merge_small_kernel<4>,
                                        (unsigned)((parents + per - 1) / per), kMergeThreads, s, m,
                                        log_g));
    }
    m.parts = (int32_t)std::max<int64_t>(
        1, std::min((f * f + kRunChildren - 1) / kRunChildren, kMergeMaxGrid / parents));
    m.parts = (int32_t)((f * f + part_children(f, m.parts) - 1) / part_children(f, m.parts));
    if (m.parts == 1)
        return hip_status(launch_kernel(&merge_kernel, (unsigned)parents, kMergeThreads, s, m));
    std::unique_lock<std::mutex> lock(g_ws_mutex, std::defer_lock);
    bool local = capturing(s);
    if (!local) {
        SplitNeed need;
        need.cnt_bytes = (size_t)(parents * kLine);
        need.part_bytes = (size_t)(parents * m.parts * kLine);
        lock.lock();
        local = !own_workspace(s, need, &m.ws);
        if (local) lock.unlock();
    }
    if (local)
        return hip_status(launch_with_lds(&merge_local_kernel, (unsigned)parents,
                                          kMergeLocalThreads, (size_t)m.parts * 4 * sizeof(float4),
                                          s, m));
    return hip_status(launch_kernel(&merge_kernel, (unsigned)(parents * m.parts), kMergeThreads, s,
                                    m));
}

iqa_status check_common(const float *x, const float *y, int64_t N, int64_t NT) {
    if (!x || !y) return IQA_ERR_NULL;
    iqa_status st = check_shape(N, NT);
    if (st != IQA_OK) return st;
    if (!aligned(x, 4) || !aligned(y, 4)) return IQA_ERR_ALIGN;
    return IQA_OK;
}

iqa_status check_outputs_params(float *lisi, float *auglisi, float *sums, float D, float C1,
                                float C2, float C) {
    if (!lisi && !auglisi && !sums) return IQA_ERR_NULL;
    if (!aligned(lisi, 4) || !aligned(auglisi, 4) || !aligned(sums, 16)) return IQA_ERR_ALIGN;
    const bool need_l = lisi || sums, need_a = auglisi || sums;
    if (need_l && (!param_ok(D) || !param_ok(C1) || !param_ok(C2))) return IQA_ERR_PARAM;
    if (need_a && !param_ok(C)) return IQA_ERR_PARAM;
    return IQA_OK;
}

// Workgroups of a batch launch: as many as `waves` gives, but no more than one
// per unit of the XCD with the most, and than HIP launches (fewer than 2^32 work
// items); they share what is left.
constexpr int64_t kMostBlocks = UINT32_MAX / (kBatchWaves * kWave) / kXcds * kXcds;

int64_t batch_grid(int64_t waves, int64_t units) {
    const int64_t all = (units + kXcds - 1) / kXcds * kXcds;
    return std::min({waves / kBatchWaves, units < kXcds ? units : all, kMostBlocks});
}

template <int CAP>
iqa_status launch_inline(const void *descs_host, int64_t count, int64_t total_units,
                         int64_t blocks, hipStream_t s) {
    InlineDescs<CAP> in;
    std::memset(&in, 0, sizeof(in));
    std::memcpy(in.d, descs_host, (size_t)count * sizeof(BatchDesc));
    in.units = total_units;
    in.count = (int32_t)count;
    return hip_status(launch_kernel(&batch_kernel_inline<kBatchUnroll, CAP>, (unsigned)blocks,
                                    kBatchWaves * kWave, s, in));
}

}  // namespace iqa

using namespace iqa;

extern "C" {

iqa_status iqa_tiles_cfg(const float *x, const float *y, int64_t N, int64_t NT, float D,
                         float C1, float C2, float C, float *lisi, float *auglisi, float *sums,
                         const iqa_launch_cfg *cfg, void *stream) {
    iqa_status st = check_common(x, y, N, NT);
    if (st != IQA_OK) return st;
    st = check_outputs_params(lisi, auglisi, sums, D, C1, C2, C);
    if (st != IQA_OK) return st;
    return run(x, y, N, NT, D, C1, C2, C, lisi, auglisi, sums, cfg, stream, Ws::kLibrary);
}

iqa_status iqa_tiles(const float *x, const float *y, int64_t N, int64_t NT, float D, float C1,
                     float C2, float C, float *lisi, float *auglisi, float *sums, void *stream) {
    return iqa_tiles_cfg(x, y, N, NT, D, C1, C2, C, lisi, auglisi, sums, nullptr, stream);
}

iqa_status iqa_tiles_noalloc(const float *x, const float *y, int64_t N, int64_t NT, float D,
                             float C1, float C2, float C, float *lisi, float *auglisi, float *sums,
                             const iqa_launch_cfg *cfg, void *stream) {
    iqa_status st = check_common(x, y, N, NT);
    if (st != IQA_OK) return st;
    st = check_outputs_params(lisi, auglisi, sums, D, C1, C2, C);
    if (st != IQA_OK) return st;
    return run(x, y, N, NT, D, C1, C2, C, lisi, auglisi, sums, cfg, stream, Ws::kScratch);
}

iqa_status iqa_tiles_timeline(const float *x, const float *y, int64_t N, int64_t NT, float D,
                              float C1, float C2, float C, float *lisi, float *auglisi,
                              float *sums, const iqa_launch_cfg *cfg, uint64_t *stamps,
                              int64_t stamp_count, void *stream) {
    iqa_status st = check_common(x, y, N, NT);
    if (st != IQA_OK) return st;
    st = check_outputs_params(lisi, auglisi, sums, D, C1, C2, C);
    if (st != IQA_OK) return st;
    if (!stamps) return IQA_ERR_NULL;
    if (!aligned(stamps, 8)) return IQA_ERR_ALIGN;
    iqa_launch_cfg c = cfg ? *cfg : pick_cfg(N, NT, x, y);
    // One row of stamps per workgroup that a workspace-free launch would have.
    if (!cfg && c.ksplit > 1 && !tuned_or_prepared(N, NT, c, x, y)) c.ksplit = 1;
    Geometry g{};
    st = geometry(N, NT, c, g);
    if (st != IQA_OK) return st;
    if (stamp_count < 8 * g.grid) return IQA_ERR_SHAPE;
    return run(x, y, N, NT, D, C1, C2, C, lisi, auglisi, sums, &c, stream, Ws::kLibrary, stamps);
}

int64_t iqa_launch_workgroups(int64_t N, int64_t NT, const iqa_launch_cfg *cfg) {
    if (!cfg || check_shape(N, NT) != IQA_OK) return -1;
    Geometry g{};
    if (geometry(N, NT, *cfg, g) != IQA_OK) return -1;
    return g.grid;
}

iqa_status lisi_tiles(const float *x, const float *y, int64_t N, int64_t NT, float D, float C1,
                      float C2, float *lisi, void *stream) {
    iqa_status st = check_common(x, y, N, NT);
    if (st != IQA_OK) return st;
    if (!lisi) return IQA_ERR_NULL;
    if (!aligned(lisi, 4)) return IQA_ERR_ALIGN;
    if (!param_ok(D) || !param_ok(C1) || !param_ok(C2)) return IQA_ERR_PARAM;
    return run(x, y, N, NT, D, C1, C2, 1.0f, lisi, nullptr, nullptr, nullptr, stream,
               Ws::kLibrary);
}

iqa_status auglisi_tiles(const float *x, const float *y, int64_t N, int64_t NT, float C,
                         float *auglisi, void *stream) {
    iqa_status st = check_common(x, y, N, NT);
    if (st != IQA_OK) return st;
    if (!auglisi) return IQA_ERR_NULL;
    if (!aligned(auglisi, 4)) return IQA_ERR_ALIGN;
    if (!param_ok(C)) return IQA_ERR_PARAM;
    return run(x, y, N, NT, 1.0f, 1.0f, 1.0f, C, nullptr, auglisi, nullptr, nullptr, stream,
               Ws::kLibrary);
}

iqa_status iqa_default_cfg(int64_t N, int64_t NT, const float *x, const float *y,
                           iqa_launch_cfg *cfg) {
    if (!cfg) return IQA_ERR_NULL;
    iqa_status st = check_shape(N, NT);
    if (st != IQA_OK) return st;
    *cfg = pick_cfg(N, NT, x, y);
    return IQA_OK;
}

iqa_status iqa_check_cfg(int64_t N, int64_t NT, const iqa_launch_cfg *cfg) {
    if (!cfg) return IQA_ERR_NULL;
    iqa_status st = check_shape(N, NT);
    if (st != IQA_OK) return st;
    Geometry g{};
    return geometry(N, NT, *cfg, g);
}

iqa_status iqa_prepare(int64_t N, int64_t NT, const iqa_launch_cfg *cfg, void *stream) {
    iqa_status st = check_shape(N, NT);
    if (st != IQA_OK) return st;
    // The default shape, and so its parts, depends on how the images are
    // aligned: what it needs at 16, 8 and 4 bytes.
    for (uintptr_t at : {256, 264, 260}) {
        const float *probe = reinterpret_cast<const float *>(at);
        st = run(probe, probe, N, NT, 1.f, 1.f, 1.f, 1.f, nullptr, nullptr, nullptr, cfg, stream,
                 Ws::kPrepare);
        if (st != IQA_OK || cfg) return st;
    }
    return IQA_OK;
}

iqa_status iqa_tune_set(int64_t N, int64_t NT, int kind, const iqa_launch_cfg *cfg) {
    if (!cfg) return IQA_ERR_NULL;
    // N == 0 registers the entry for every image size with this tile size.
    iqa_status st = check_shape(N == 0 ? NT : N, NT);
    if (st != IQA_OK) return st;
    if (kind != IQA_TUNE_SINGLE && kind != IQA_TUNE_BATCH && kind != IQA_TUNE_SERVE)
        return IQA_ERR_CONFIG;
    Geometry g{};
    st = geometry(N == 0 ? NT : N, NT, *cfg, g);
    if (st != IQA_OK) return st;
    if (cfg->vec != 4) return IQA_ERR_CONFIG;
    if (kind != IQA_TUNE_SINGLE && !batch_geometry_ok(*cfg)) return IQA_ERR_CONFIG;
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    g_tuned[std::make_tuple(N, NT, kind)] = *cfg;
    return IQA_OK;
}

void iqa_tune_clear(void) {
    std::lock_guard<std::mutex> lock(g_tune_mutex);
    g_tuned.clear();
}

int64_t iqa_batch_default_waves(void) {
    return kTunedBatchWaves > 0 ? kTunedBatchWaves : 2048;
}

iqa_status iqa_batch_cfg(int64_t N, int64_t NT, iqa_launch_cfg *cfg) {
    if (!cfg) return IQA_ERR_NULL;
    iqa_status st = check_shape(N, NT);
    if (st != IQA_OK) return st;
    if (NT % 4 != 0) return IQA_ERR_CONFIG;
    *cfg = batch_cfg(N, NT);
    return IQA_OK;
}

iqa_status iqa_serve_cfg(int64_t N, int64_t NT, iqa_launch_cfg *cfg) {
    if (!cfg) return IQA_ERR_NULL;
    iqa_status st = check_shape(N, NT);
    if (st != IQA_OK) return st;
    if (NT % 4 != 0) return IQA_ERR_CONFIG;
    *cfg = serve_cfg(N, NT);
    return IQA_OK;
}

iqa_status iqa_batch_describe(const iqa_pair *pairs, int64_t count, void *descs,
                              int64_t *total_units) {
    return iqa::describe_pairs(pairs, count, descs, total_units, IQA_TUNE_BATCH);
}

iqa_status iqa_odd_batch_describe(const iqa_pair *pairs, int64_t count, void *descs,
                                  int64_t *total_units) {
    return iqa::describe_pairs(pairs, count, descs, total_units, iqa::kDescribeOdd);
}

}  // extern "C"

iqa_status iqa::describe_pairs(const iqa_pair *pairs, int64_t count, void *descs,
                               int64_t *total_units, int kind) {
    if (!pairs || !descs || !total_units) return IQA_ERR_NULL;
    if (count < 1 || count > INT_MAX) return IQA_ERR_SHAPE;
    BatchDesc *out = static_cast<BatchDesc *>(descs);
    int64_t units = 0;
    for (int64_t i = 0; i < count; ++i) {
        const iqa_pair &p = pairs[i];
        iqa_status st = check_common(p.x, p.y, p.N, p.NT);
        if (st != IQA_OK) return st;
        st = check_outputs_params(p.lisi, p.auglisi, p.sums, p.D, p.C1, p.C2, p.C);
        if (st != IQA_OK) return st;
        const bool odd = kind == kDescribeOdd;
        if (!odd && p.NT % 4 != 0) return IQA_ERR_CONFIG;
        const uintptr_t unit = odd ? 4 : 16;
        if (!aligned(p.x, unit) || !aligned(p.y, unit)) return IQA_ERR_ALIGN;
        const iqa_launch_cfg c = odd                      ? pick_cfg(p.N, p.NT, p.x, p.y)
                                 : kind == IQA_TUNE_SERVE ? serve_cfg(p.N, p.NT)
                                                          : batch_cfg(p.N, p.NT);
        Geometry g{};
        st = geometry(p.N, p.NT, c, g);
        if (st != IQA_OK) return st;
        if (odd && (!g.any || c.ksplit != 1)) return IQA_ERR_CONFIG;
        BatchDesc d;
        std::memset(&d, 0, sizeof(d));
        // Outputs a pair does not ask for stay NULL; the batch always computes
        // all four sums, so lisi and auglisi get the constants they need.
        fill_pair(d.a, p.x, p.y, p.N, p.NT, p.lisi || p.sums ? p.D : 1.f,
                  p.lisi || p.sums ? p.C1 : 1.f, p.lisi || p.sums ? p.C2 : 1.f,
                  p.auglisi || p.sums ? p.C : 1.f, p.lisi, p.auglisi, p.sums, c, g);
        d.unit_begin = units;
        units += odd ? g.groups : batch_units(d.a);
        std::memcpy(out + i, &d, sizeof(d));
    }
    if (units > ((int64_t)1 << 40)) return IQA_ERR_SHAPE;
    *total_units = units;
    return IQA_OK;
}

extern "C" {

iqa_status iqa_tiles_batched(const void *descs_dev, int64_t count, int64_t total_units,
                             int64_t waves, void *stream) {
    if (!descs_dev) return IQA_ERR_NULL;
    if (count < 1 || count > INT_MAX || total_units < 1) return IQA_ERR_SHAPE;
    if (!aligned(descs_dev, 16)) return IQA_ERR_ALIGN;
    if (waves < kBatchWaves || waves % kBatchWaves != 0 || waves / kBatchWaves > INT_MAX)
        return IQA_ERR_CONFIG;
    const int64_t blocks = batch_grid(waves, total_units);
    return hip_status(launch_kernel(&batch_kernel<kBatchUnroll>, (unsigned)blocks,
                                    kBatchWaves * kWave, static_cast<hipStream_t>(stream),
                                    static_cast<const BatchDesc *>(descs_dev), (int)count,
                                    total_units));
}

iqa_status iqa_odd_tiles_batched(const void *descs_dev, int64_t count, int64_t total_units,
                                 void *stream) {
    if (!descs_dev) return IQA_ERR_NULL;
    if (count < 1 || count > INT_MAX || total_units < 1) return IQA_ERR_SHAPE;
    if (!aligned(descs_dev, 16)) return IQA_ERR_ALIGN;
    const int64_t blocks = batch_grid(kMostBlocks * kBatchWaves, total_units);
    return hip_status(launch_kernel(&odd_batch_kernel, (unsigned)blocks, kBatchWaves * kWave,
                                    static_cast<hipStream_t>(stream),
                                    static_cast<const BatchDesc *>(descs_dev), (int)count,
                                    total_units));
}

iqa_status iqa_tiles_batched_inline(const void *descs_host, int64_t count, int64_t total_units,
                                    int64_t waves, void *stream) {
    if (!descs_host) return IQA_ERR_NULL;
    if (count > IQA_BATCH_INLINE_MAX) return IQA_ERR_SHAPE;
    return iqa::tiles_batched_args(descs_host, count, total_units, waves, stream);
}

}  // extern "C"

iqa_status iqa::tiles_batched_args(const void *descs_host, int64_t count, int64_t total_units,
                                   int64_t waves, void *stream) {
    if (count < 1 || count > kArgsMax || total_units < 1) return IQA_ERR_SHAPE;
    if (waves < kBatchWaves || waves % kBatchWaves != 0 || waves / kBatchWaves > INT_MAX)
        return IQA_ERR_CONFIG;
    // The table is on the host here, so its unit numbering is checked: pair i
    // starts where pair i - 1 ends, and the pairs cover exactly total_units.
    int64_t next = 0;
    for (int64_t i = 0; i < count; ++i) {
        BatchDesc d;
        std::memcpy(&d, static_cast<const BatchDesc *>(descs_host) + i, sizeof(d));
        if (d.unit_begin != next || d.a.ns < 1 || d.a.ngx < 1) return IQA_ERR_CONFIG;
        next += batch_units(d.a);
    }
    if (next != total_units) return IQA_ERR_CONFIG;
    const int64_t blocks = batch_grid(waves, total_units);
    const hipStream_t s = static_cast<hipStream_t>(stream);
    if (count == 1) return launch_inline<1>(descs_host, count, total_units, blocks, s);
    if (count <= 4) return launch_inline<4>(descs_host, count, total_units, blocks, s);
    if (count <= IQA_BATCH_INLINE_MAX)
        return launch_inline<IQA_BATCH_INLINE_MAX>(descs_host, count, total_units, blocks, s);
    return launch_inline<kArgsMax>(descs_host, count, total_units, blocks, s);
}

extern "C" {

iqa_status iqa_merge_tiles(const float *sums_in, int64_t ns, int64_t f, float D, float C2,
                           float C, float *lisi, float *auglisi, float *sums_out, void *stream) {
    if (!sums_in) return IQA_ERR_NULL;
    if (ns <= 0 || f <= 0 || ns % f != 0 || ns > IQA_MAX_N) return IQA_ERR_SHAPE;
    iqa_status st = check_outputs_params(lisi, auglisi, sums_out, D, 1.f, C2, C);
    if (st != IQA_OK) return st;
    if (!aligned(sums_in, 16)) return IQA_ERR_ALIGN;
    const int64_t np = ns / f;
    if (np * np > INT_MAX) return IQA_ERR_SHAPE;
    return merge(sums_in, ns, f, D, C2, C, lisi, auglisi, sums_out,
                 static_cast<hipStream_t>(stream));
}

iqa_status iqa_pyramid(const float *sums_in, int64_t ns, int64_t levels, float D, float C2, float C,
                       float *const *lisi, float *const *auglisi, float *const *sums_out,
                       void *stream) {
    if (!sums_in) return IQA_ERR_NULL;
    if (ns <= 0 || ns > IQA_MAX_N || levels < 1 || levels > 17 || ns % (int64_t(1) << levels) != 0)
        return IQA_ERR_SHAPE;
    if ((ns / 2) * (ns / 2) > INT_MAX) return IQA_ERR_SHAPE;   // as a merge of the first level
    if (!lisi || !auglisi || !sums_out) return IQA_ERR_NULL;
    if (!aligned(sums_in, 16)) return IQA_ERR_ALIGN;
    for (int64_t l = 0; l < levels; ++l) {
        const iqa_status st = check_outputs_params(lisi[l], auglisi[l], sums_out[l], D, 1.f, C2, C);
        if (st != IQA_OK) return st;
        // The sums of every sixth level feed the next launch.
        if ((l + 1) % kPyramidLevels == 0 && l + 1 < levels && !sums_out[l]) return IQA_ERR_NULL;
    }
    for (int64_t l = 0; l < levels; l += kPyramidLevels) {
        PyramidArgs a{};
        a.sums_in = l ? sums_out[l - 1] : sums_in;
        a.ns = (int32_t)(ns >> l);
        a.levels = (int32_t)std::min<int64_t>(kPyramidLevels, levels - l);
        a.nbx = (a.ns + 63) / 64;
        a.D = D;
        a.C2 = C2;
        a.C = C;
        for (int i = 0; i < a.levels; ++i) {
            a.lisi[i] = lisi[l + i];
            a.aug[i] = auglisi[l + i];
            a.sums[i] = sums_out[l + i];
        }
        const iqa_status st =
            hip_status(launch_kernel(&pyramid_kernel, (unsigned)(a.nbx * a.nbx), kPyramidThreads,
                                     static_cast<hipStream_t>(stream), a));
        if (st != IQA_OK) return st;
    }
    return IQA_OK;
}

iqa_status iqa_read_ceiling(const float *buf, int64_t n, float *out, int64_t blocks,
                            void *stream) {
    if (!buf || !out) return IQA_ERR_NULL;
    if (n <= 0 || n % 4 != 0 || blocks <= 0 || blocks > INT_MAX) return IQA_ERR_SHAPE;
    if (!aligned(buf, 16) || !aligned(out, 4)) return IQA_ERR_ALIGN;
    const int64_t n4 = n / 4;
    const int64_t per = (n4 + blocks - 1) / blocks;
    return hip_status(launch_kernel(&read_ceiling_kernel, (unsigned)blocks, 256,
                                    static_cast<hipStream_t>(stream),
                                    reinterpret_cast<const float4 *>(buf), n4, per, out));
}

const char *iqa_status_str(int status) {
    switch (status) {
        case IQA_OK: return "IQA_OK";
        case IQA_ERR_NULL: return "IQA_ERR_NULL: a required pointer is NULL or no output was requested";
        case IQA_ERR_SHAPE: return "IQA_ERR_SHAPE: N and NT must be positive, NT must divide N, N <= 2^17";
        case IQA_ERR_ALIGN: return "IQA_ERR_ALIGN: a float pointer is not 4-byte aligned (sums: 16-byte)";
        case IQA_ERR_PARAM: return "IQA_ERR_PARAM: D, C1, C2 and C must be positive, finite, normal floats";
        case IQA_ERR_HIP: return "IQA_ERR_HIP: a HIP call or kernel launch failed";
        case IQA_ERR_CONFIG: return "IQA_ERR_CONFIG: launch configuration invalid for this shape";
        case IQA_ERR_CAPTURE: return "IQA_ERR_CAPTURE: workspace must grow while the stream is captured";
        case IQA_ERR_BUDGET: return "IQA_ERR_BUDGET: the request can never fit the server's HBM budget";
        case IQA_ERR_TIMEOUT: return "IQA_ERR_TIMEOUT: the wait ran out of time";
        case IQA_ERR_SCRATCH: return "IQA_ERR_SCRATCH: the shape needs more split scratch than iqa_tiles_noalloc holds";
        default: return "unknown iqa_status";
    }
}

int iqa_last_hip_error(void) { return g_last_hip_error; }

int iqa_version(void) { return 400; }

}  // extern "C"
