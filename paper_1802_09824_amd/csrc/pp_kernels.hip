// The PP (particle-particle) kernels: short-range pair sums over the block
// lists, FP32 (the hot path), FP64 (the yardstick) and an FP64 pair count.
//
// Per pair (sec. 3.1, Eq. equ:split, with Plummer softening):
//   a_i += G m_j d g(s_eps / 2 r_s) / s_eps^3,   kept iff s < r_cut.
// FP32 form.  Lengths are in units of ell = 2 r_s sqrt(U_MAX / 2),
// relative to the FP64 centre of the target block (the origin subtraction
// is done in FP64 when a source is staged, so the FP32 offsets are small
// and precise).  With g(x) = 1 - x^3 H(x^2), H a polynomial fitted on
// u = x^2 in [0, U_MAX] in the variable t = 2u / U_MAX - 1 (split_poly.h),
// r2 = s_eps^2 / ell^2 and y = 1 / sqrt(r2) (hardware reciprocal square
// root), the unit makes t = r2 - 1 and
//   ell^3 g / s_eps^3 = y^3 - (U_MAX / 2)^(3/2) H(u),
// so the polynomial's coefficients are the same literals for every box and
// G / ell^2 scales the sum at the end.  Softening enters r2 through the
// first fused multiply-add; the cut test compares r2 with
// (r_cut^2 + eps^2) / ell^2.  Every operand of the pair arithmetic is a
// VGPR or a literal: on gfx950 two waves' VALU instructions issue together
// only then.
// Sources are staged 64 at a time in LDS and broadcast to the 64 lanes
// (one target per lane).  Each tile of 64 pairs is summed in FP32 and the
// tile sums enter a Kahan-compensated per-target total.  Work items are
// (target block, chunk of its source list); their partial sums are reduced
// in FP64 in a fixed order, so results do not depend on scheduling.
#include <cmath>

#include "pp_internal.h"
#include "split_poly.h"
#include "split_poly64.h"

namespace pp {
namespace {

struct ItemArgs {
    const int32_t* iblock;
    const int32_t* is0;
    const int32_t* is1;
    const int64_t* sizes;      // the counts of the lists (SizeSlot), on the device
    const int32_t* bstart;
    const int32_t* bcount;
    const IBox* bbox;
    const int32_t* bboxid;
    const int64_t* roff;
    const int32_t* rbeg;
    const int32_t* rpre;
    const uint8_t* rcode;
    const int64_t* ioff;
    const BoxDev* box;
    const int32_t* perm;       // key order -> input order
    const int32_t* mass_flag;  // per box: 1 where the masses are not all equal
    const float4* split_tab;   // the interpolated split table (variant bit 8)
    float* acc;                // FP32 output (single-item blocks write it directly)
    int wide;                  // acc: a 16-byte record per particle (Work::acc_wide), else three rows
    const uint8_t* active;     // per input particle: outputs written only where set (null: all)
    const uint64_t* bact;      // per block: the lanes whose targets are active (set with active)
};

// Particle i's result.
__device__ __forceinline__ void put_acc(float* __restrict__ acc, int wide, int64_t N, int64_t i, float x, float y,
                                        float z) {
    if (wide) {
        reinterpret_cast<float4*>(acc)[i] = make_float4(x, y, z, 0.f);
    } else {
        acc[i] = x;
        acc[N + i] = y;
        acc[2 * N + i] = z;
    }
}

__device__ __forceinline__ bool target_on(const ItemArgs& ia, int64_t i) {
    return !ia.active || ia.active[i] != 0;
}

ItemArgs item_args(const BatchDev& bd, const Work& w) {
    ItemArgs ia;
    ia.iblock = w.iblock.as<int32_t>();
    ia.is0 = w.is0.as<int32_t>();
    ia.is1 = w.is1.as<int32_t>();
    ia.sizes = w.sizes.as<int64_t>();
    ia.bstart = w.bstart.as<int32_t>();
    ia.bcount = w.bcount.as<int32_t>();
    ia.bbox = w.bbox.as<IBox>();
    ia.bboxid = w.bboxid.as<int32_t>();
    ia.roff = w.roff.as<int64_t>();
    ia.rbeg = w.rbeg.as<int32_t>();
    ia.rpre = w.rpre.as<int32_t>();
    ia.rcode = w.rcode.as<uint8_t>();
    ia.ioff = w.ioff.as<int64_t>();
    ia.box = bd.box;
    ia.perm = w.perm.as<int32_t>();
    ia.mass_flag = w.mass_flag.as<int32_t>();
    ia.split_tab = w.split_tab.as<float4>();
    ia.acc = nullptr;
    ia.wide = w.acc_wide;
    ia.active = w.active;
    ia.bact = w.active ? w.bact.as<uint64_t>() : nullptr;
    return ia;
}

// The item of a workgroup of the one-workgroup-per-item launches, or -1 for
// one past the end.  The 8 XCDs take workgroups round-robin; each gets
// stretches of kStretch consecutive items, every eighth one: neighbouring
// target blocks share most of their sources, which then stay in that XCD's
// L2, and dense regions are dealt out over all XCDs.  One long stretch per
// XCD left the XCDs with the dense regions running alone at the end: 2.1 M
// clustered particles took 6.63 ms where stretches of 16 to 256 take 6.02 to
// 6.10 (a uniform box does not care: 2.93 to 2.96 ms).
constexpr int64_t kStretch = 64;

__device__ __forceinline__ int64_t xcd_item(int64_t bid, int64_t nitem) {
    const int64_t k = bid >> 3;
    const int64_t item = ((k / kStretch) * 8 + (bid & 7)) * kStretch + k % kStretch;
    return item < nitem ? item : -1;
}

// The workgroups such a launch needs for n items.
int64_t xcd_groups(int64_t n) { return (n + 8 * kStretch - 1) / (8 * kStretch) * (8 * kStretch); }

__device__ __forceinline__ int64_t find_range(const int32_t* __restrict__ rpre, int64_t lo,
                                              int64_t hi, int32_t p) {
    // last r in [lo, hi] with rpre[r] <= p (rpre ascending, rpre[lo] <= p)
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (rpre[mid] <= p) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// The same search by a whole wave, for a wave-uniform p: each round reads
// 64 evenly spaced entries and keeps the stretch between two of them, so
// the dependent loads number log_64 of the range count instead of log_2.
__device__ __forceinline__ int64_t find_range_wave(const int32_t* __restrict__ rpre, int64_t lo,
                                                   int64_t hi, int32_t p) {
    const int lane = threadIdx.x & 63;
    while (lo < hi) {
        const int64_t stride = (hi - lo + 64) / 64;   // ceil((hi - lo + 1) / 64)
        const int64_t q = lo + lane * stride;
        const bool le = q <= hi && rpre[q] <= p;
        const int c = __popcll(__ballot(le));        // >= 1: rpre[lo] <= p
        lo += (int64_t)(c - 1) * stride;
        const int64_t top = lo + stride - 1;
        hi = top < hi ? top : hi;
        if (stride == 1) break;
    }
    return lo;
}

constexpr double csqrt(double x) {
    double r = x > 1.0 ? x : 1.0;
    for (int i = 0; i < 64; ++i) r = 0.5 * (r + x / r);
    return r;
}
// (U_MAX / 2)^(3/2): H's factor in the length unit ell
constexpr double kHScale = 0.5 * SPLIT_POLY_U_MAX * csqrt(0.5 * SPLIT_POLY_U_MAX);
// H's coefficients times (U_MAX / 2)^(3/2), rounded once to FP32: the pair
// loop's literal operands
struct HCoef {
    float c[SPLIT_POLY_DEGREE + 1];
};
constexpr HCoef make_hcoef() {
    HCoef h{};
    for (int j = 0; j <= SPLIT_POLY_DEGREE; ++j) h.c[j] = (float)(kHScale * SPLIT_POLY_C[j]);
    return h;
}
constexpr HCoef kHC = make_hcoef();

// (U_max/2)^{3/2} H(u) at r2 = s_eps^2 / ell^2: the polynomial in t = r2 - 1
// (Horner, one FMA per degree), or (TABLE) the interpolated table of the
// paper's design: kTabN quadratic pieces over r2 in [0, 2), each stored as
// (a, b, c) with h = a + z (b + z c), z the position inside the piece.  Past r2 = 2 the
// last piece is extrapolated; such pairs lie beyond the cut and are masked.
constexpr int kTabN = 128;

template <bool TABLE>
__device__ __forceinline__ float split_h(float r2, const float4* __restrict__ tab) {
    if (TABLE) {
        const float sidx = r2 * (float)(kTabN / 2);
        int k = (int)sidx;
        k = k < kTabN - 1 ? k : kTabN - 1;
        const float z = sidx - (float)k;
        const float4 c = tab[k];
        return fmaf(fmaf(c.z, z, c.y), z, c.x);
    }
    const float t = r2 - 1.f;
    float h = kHC.c[SPLIT_POLY_DEGREE];
#pragma unroll
    for (int j = SPLIT_POLY_DEGREE - 1; j >= 0; --j) h = fmaf(h, t, kHC.c[j]);
    return h;
}

// One source against the lane's target; adds into (tx, ty, tz).
template <bool NEWTON, bool TABLE = false>
__device__ __forceinline__ void pair_f32(const float4 sj, float xi, float yi, float zi,
                                         const PolyF32& P, float& tx, float& ty, float& tz,
                                         const float4* __restrict__ tab = nullptr) {
    const float dx = sj.x - xi, dy = sj.y - yi, dz = sj.z - zi;
    float r2 = fmaf(dx, dx, P.eps2n);
    r2 = fmaf(dy, dy, r2);
    r2 = fmaf(dz, dz, r2);
    float y = __builtin_amdgcn_rsqf(r2);
    if (NEWTON) y = y * fmaf(-0.5f * r2 * y, y, 1.5f);
    const float h = split_h<TABLE>(r2, tab);
    float F = fmaf(y * y, y, -h) * sj.w;
    F = r2 < P.cut2 ? F : 0.f;
    tx = fmaf(F, dx, tx);
    ty = fmaf(F, dy, ty);
    tz = fmaf(F, dz, tz);
}

// The same for a box whose masses are all equal: the source's w slot holds
// the cut on r2 instead of the mass (which joins the final scale), so the
// tile keeps its 16-byte entries and the mass multiply drops out.
template <bool NEWTON, bool TABLE = false>
__device__ __forceinline__ void pair_f32_eq(const float4 sj, float xi, float yi, float zi,
                                            float& tx, float& ty, float& tz, float eps2,
                                            const float4* __restrict__ tab = nullptr) {
    const float dx = sj.x - xi, dy = sj.y - yi, dz = sj.z - zi;
    float r2 = fmaf(dx, dx, eps2);
    r2 = fmaf(dy, dy, r2);
    r2 = fmaf(dz, dz, r2);
    float y = __builtin_amdgcn_rsqf(r2);
    if (NEWTON) y = y * fmaf(-0.5f * r2 * y, y, 1.5f);
    const float h = split_h<TABLE>(r2, tab);
    float F = fmaf(y * y, y, -h);
    F = r2 < sj.w ? F : 0.f;
    tx = fmaf(F, dx, tx);
    ty = fmaf(F, dy, ty);
    tz = fmaf(F, dz, tz);
}

__device__ __forceinline__ void kahan_add(float& s, float& c, float v) {
    const float y = v - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

__device__ __forceinline__ float readlane_f(float v, int lane) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

__device__ __forceinline__ int64_t readlane64(int64_t v, int lane) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// The ranges of the 64 list positions from `base` on (positions below s1),
// one position per lane: its range r, that range's first particle, list
// position and shift code.  rcur: a range at or before the one that holds
// `base`, at most K * 64 positions before it.  A window inside the range at
// the cursor needs no mapping; otherwise the wave reads the 64 ranges from the
// cursor on (one per lane), marks in LDS the window positions where one of
// them starts, and each lane takes its position's range from the count of
// marks up to it and the range's first particle from the lane that read it;
// only a window that runs past those 64 ranges falls back to a binary search
// per lane.
template <int K>
__device__ __forceinline__ int64_t window_range(const ItemArgs& ia, int32_t base, int32_t s1, int64_t rcur,
                                                int64_t r_hi, int* mark, int32_t& rb, int32_t& rp,
                                                int& code) {
    const int lane = threadIdx.x & (kBlock - 1);
    const int32_t p = base + lane;
    const int32_t last = s1 - 1 < base + kBlock - 1 ? s1 - 1 : base + kBlock - 1;
    int64_t r;
    // the block's last range: every position of the item lies before its end
    const int32_t end_cur = rcur < r_hi ? ia.rpre[rcur + 1] : s1;
    if (last < end_cur) {
        // the cursor's range holds the whole window: nothing to map
        r = rcur;
        rb = ia.rbeg[rcur];
        rp = ia.rpre[rcur];
        code = ia.rcode[rcur];
    } else {
        // the ranges rcur .. rcur + 63, one per lane
        const int64_t rq = rcur + lane;
        const bool rv = rq <= r_hi;
        const int32_t qpre = rv ? ia.rpre[rq] : INT32_MAX;
        const int32_t qbeg = rv ? ia.rbeg[rq] : 0;
        const int qcode = rv ? (int)ia.rcode[rq] : 13;
        // ranges that start at or before the window's first (last) position
        const int c0 = __popcll(__ballot(qpre <= base));
        const int c1 = __popcll(__ballot(qpre <= last));
        if (c1 < kBlock || rcur + (kBlock - 1) >= r_hi) {
            // every range of the window was read: mark where they start
            mark[lane] = 0;
            wave_sync();
            if (qpre > base && qpre <= last) mark[qpre - base] = 1;
            wave_sync();
            const uint64_t starts = __ballot(mark[lane] != 0);
            wave_sync();
            const uint64_t upto = lane == 63 ? ~0ull : (2ull << lane) - 1ull;
            const int idx = c0 - 1 + __popcll(starts & upto);
            rb = __shfl(qbeg, idx);
            rp = __shfl(qpre, idx);
            code = __shfl(qcode, idx);
            r = rcur + idx;
        } else {
            // more than 64 ranges in reach: the window starts at most K * 64
            // positions (so ranges) past the cursor's
            const int64_t top = rcur + K * kBlock < r_hi ? rcur + K * kBlock : r_hi;
            r = p < s1 ? find_range(ia.rpre, rcur, top, p) : rcur;
            rb = ia.rbeg[r];
            rp = ia.rpre[r];
            code = ia.rcode[r];
        }
    }
    return r;
}

// One work item of the FP32 PP kernel on one wave (target block, chunk of
// its source list).  Sources are fetched 64 list positions at a time (their
// ranges by window_range).  Each lane loads
// the FP64 position and the mass; the loads of the next window are issued
// before the current tile is swept.  A fetched source is shifted by its periodic image, made
// relative to the FP64 block centre, scaled by 1/ell and rounded to FP32,
// and dropped if it lies at r_cut or more from each of the four boxes
// around the block's runs of 16 targets.  Survivors are compacted with a
// ballot into a 128-entry LDS ring; every 64 survivors are swept by all
// lanes with broadcast LDS reads.
//
// K waves may share one item (the workgroup is K waves): wave k takes the
// windows k, k + K, k + 2K, ... of the item's list, stages and sweeps them
// into its own LDS ring and its own compensated sums, and the K sums are
// added in wave order in FP64 (through LDS) before the item's result is
// written.  The split does not depend on scheduling, so results stay
// reproducible for a given K.
//
// PACK (calls with active flags): a block with at most 32 (16) active targets
// holds them 2 (4) times in the wave, each copy sweeping its own tile of 64
// staged sources at the same time; the copies' tile sums then enter the
// compensated totals one after the other, in tile order.  Staging, tiles and
// sums are those of the whole block, so the results are bit-identical to it,
// at half (a quarter) of the sweeps.  On 2.1 M clustered particles with 40 %
// of the sphere members active a whole call went from 6.38 to 4.19 ms, on 1 M
// with reused lists from 2.27 to 1.42.
constexpr int kPackMax = 4;            // copies at most
// tile entries per wave: the copies' tiles and the ring's slack, each stretch
// of 64 shifted by one entry so that the copies read different LDS banks
template <int VAR>
constexpr int tile_entries() { return (VAR & 16) ? (kPackMax + 1) * (kBlock + 1) : 2 * kBlock; }

// Copies (a power of two) of a block's active targets that one wave holds when
// na of them are active (pp_item, PACK).
__device__ __forceinline__ int pack_copies(int na) { return na <= kBlock / 4 ? 2 : na <= kBlock / 2 ? 1 : 0; }

template <int VAR, int K>
__device__ __forceinline__ void pp_item(const ItemArgs& ia, int64_t item,
                                        const double* __restrict__ pos_s,
                                        const float* __restrict__ mass_s, int64_t N,
                                        float* __restrict__ partial,
                                        int32_t* __restrict__ icount, float4* tile_all,
                                        const float4* __restrict__ tab, float4* qb_all,
                                        double* red, int* mark_all) {
    constexpr bool NEWTON = (VAR & 1) != 0;
    constexpr bool KAHAN = (VAR & 2) == 0;
    constexpr bool LOCAL = (VAR & 4) == 0;     // FP64 block-centre subtraction
    constexpr bool TABLE = (VAR & 8) != 0;     // interpolated split table
    constexpr bool PACK = (VAR & 16) != 0;     // several tiles at once for blocks with few active targets
    static_assert(!PACK || (KAHAN && LOCAL), "packing keeps the production arithmetic");
    const int lane = threadIdx.x & (kBlock - 1);
    const int wv = K > 1 ? (int)(threadIdx.x / kBlock) : 0;
    float4* tile = tile_all + wv * tile_entries<VAR>();
    const int32_t b = ia.iblock[item];
    const int32_t s0 = ia.is0[item];
    const int32_t s1 = ia.is1[item];
    const int32_t nt = ia.bcount[b];
    const int xbox = ia.bboxid[b];
    const BoxDev& X = ia.box[xbox];
    const double L = X.L, cell = X.cell, inv_len = X.inv_len;
    PolyF32 P = X.poly;
    // the pair loop's constants stay in VGPRs: with an SGPR operand an
    // instruction issues at half the rate
    asm("" : "+v"(P.eps2n));
    asm("" : "+v"(P.cut2));
    // equal masses (the compensated form only): the mass joins the final scale
    const bool equal = KAHAN && ia.mass_flag[xbox] == 0;
    const float mu = equal ? mass_s[X.poff] : 1.f;
    const IBox B = ia.bbox[b];
    const double ox = 0.5 * (double)(B.lo[0] + B.hi[0]) * cell;
    const double oy = 0.5 * (double)(B.lo[1] + B.hi[1]) * cell;
    const double oz = 0.5 * (double)(B.lo[2] + B.hi[2]) * cell;
    // half sides of the block box in units of ell, widened slightly so the
    // pruning test can only keep too much
    const float hx = (float)(0.5 * (double)(B.hi[0] - B.lo[0]) * cell * inv_len) * 1.0001f + 1e-6f;
    const float hy = (float)(0.5 * (double)(B.hi[1] - B.lo[1]) * cell * inv_len) * 1.0001f + 1e-6f;
    const float hz = (float)(0.5 * (double)(B.hi[2] - B.lo[2]) * cell * inv_len) * 1.0001f + 1e-6f;
    const float keep2 = P.keep2;
    const int64_t t = (int64_t)ia.bstart[b] + lane;
    float xi = 0.f, yi = 0.f, zi = 0.f;
    if (lane < nt) {
        xi = (float)((pos_s[t] - (LOCAL ? ox : 0.0)) * inv_len);
        yi = (float)((pos_s[N + t] - (LOCAL ? oy : 0.0)) * inv_len);
        zi = (float)((pos_s[2 * N + t] - (LOCAL ? oz : 0.0)) * inv_len);
    }
    // Four boxes around the FP32 offsets of the four runs of 16 consecutive
    // targets (key order), kept in LDS: a source is staged when it comes
    // within the cut of any of them, which drops about 5 % of the sources
    // that pass the whole block's box.  Widened like the block box.
    constexpr int GROUPS = 4;
    constexpr int GW = kBlock / GROUPS;
    float4* qb = qb_all + wv * 2 * GROUPS;
    if (LOCAL) {
        float ax_ = lane < nt ? xi : INFINITY, bx_ = lane < nt ? xi : -INFINITY;
        float ay_ = lane < nt ? yi : INFINITY, by_ = lane < nt ? yi : -INFINITY;
        float az_ = lane < nt ? zi : INFINITY, bz_ = lane < nt ? zi : -INFINITY;
#pragma unroll
        for (int m = 1; m < GW; m <<= 1) {
            ax_ = fminf(ax_, __shfl_xor(ax_, m));
            bx_ = fmaxf(bx_, __shfl_xor(bx_, m));
            ay_ = fminf(ay_, __shfl_xor(ay_, m));
            by_ = fmaxf(by_, __shfl_xor(by_, m));
            az_ = fminf(az_, __shfl_xor(az_, m));
            bz_ = fmaxf(bz_, __shfl_xor(bz_, m));
        }
        // an empty group repeats group 0
        {
            const bool empty = lane >= nt;
            const float r0 = readlane_f(ax_, 0), r1 = readlane_f(bx_, 0), r2 = readlane_f(ay_, 0);
            const float r3 = readlane_f(by_, 0), r4 = readlane_f(az_, 0), r5 = readlane_f(bz_, 0);
            ax_ = empty ? r0 : ax_;
            bx_ = empty ? r1 : bx_;
            ay_ = empty ? r2 : ay_;
            by_ = empty ? r3 : by_;
            az_ = empty ? r4 : az_;
            bz_ = empty ? r5 : bz_;
        }
        wave_sync();
        if (lane % GW == 0) {
            const int g = lane / GW;
            qb[2 * g] = make_float4(0.5f * (ax_ + bx_), 0.5f * (ay_ + by_), 0.5f * (az_ + bz_),
                                    0.5f * (bx_ - ax_) * 1.0001f + 1e-6f);
            qb[2 * g + 1] = make_float4(0.5f * (by_ - ay_) * 1.0001f + 1e-6f,
                                        0.5f * (bz_ - az_) * 1.0001f + 1e-6f, 0.f, 0.f);
        }
        wave_sync();
    }
    const int64_t r_lo = ia.roff[b], r_hi = ia.roff[b + 1] - 1;
    int* mark = mark_all + wv * kBlock;
    // PACK: copies of the active targets (a power of two), this lane's target
    // (a lane of the block) and the tile its copy sweeps
    int lcopies = 0, tlane = lane;
    bool mine = true;                                // this lane writes its target's result
    const float4* tl = tile;
    if (PACK) {
        const uint64_t on = ia.bact[b];
        const int na = __popcll(on);
        lcopies = pack_copies(na);
        mine = (on >> lane) & 1ull;
        if (lcopies > 0) {
            const int slot = lane & ((kBlock >> lcopies) - 1);
            const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(on >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)on, 0u));
            wave_sync();
            mark[lane] = 0;
            wave_sync();
            if (mine) mark[rank] = lane;
            wave_sync();
            tlane = mark[slot];
            wave_sync();
            xi = __shfl(xi, tlane);
            yi = __shfl(yi, tlane);
            zi = __shfl(zi, tlane);
            mine = lane < na;
            tl = tile + (lane >> (6 - lcopies)) * (kBlock + 1);
        }
    }
    const int full = kBlock << lcopies;              // staged sources that start a sweep
    float ax = 0.f, ay = 0.f, az = 0.f, cx = 0.f, cy = 0.f, cz = 0.f;
    int count = 0;                                   // staged sources (wave-uniform)
    int32_t staged = 0;
    const int32_t first = s0 + wv * kBlock;          // this wave's first window
    int64_t rcur = s1 > first ? find_range_wave(ia.rpre, r_lo, r_hi, first) : r_lo;

    double px = 0, py = 0, pz = 0;
    float pm = 0.f;
    int pc = 13;
    bool pv = false;
    auto fetch = [&](int32_t base) {
        const int32_t p = base + lane;
        pv = p < s1;
        int32_t rb, rp;
        int code;
        const int64_t r = window_range<K>(ia, base, s1, rcur, r_hi, mark, rb, rp, code);
        if (pv) {
            const int64_t j = (int64_t)rb + (p - rp);
            pc = code;
            px = pos_s[j];
            py = pos_s[N + j];
            pz = pos_s[2 * N + j];
            pm = mass_s[j];
        }
        rcur = readlane64(r, kBlock - 1);
    };
    // the tile sums of the first `tiles` copies enter the compensated totals
    // (kept alike in every copy) in tile order
    auto add_tiles = [&](int tiles, float tx, float ty, float tz) {
        if (PACK && lcopies > 0) {
            const int slot = lane & ((kBlock >> lcopies) - 1);
            for (int g = 0; g < tiles; ++g) {
                const int from = (g << (6 - lcopies)) | slot;
                kahan_add(ax, cx, __shfl(tx, from));
                kahan_add(ay, cy, __shfl(ty, from));
                kahan_add(az, cz, __shfl(tz, from));
            }
        } else {
            kahan_add(ax, cx, tx);
            kahan_add(ay, cy, ty);
            kahan_add(az, cz, tz);
        }
    };
    wave_sync();
    if (first < s1) fetch(first);
    for (int32_t base = first; base < s1; base += K * kBlock) {
        bool keep = false;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (pv) {
            const double sx = (double)(pc / 9 - 1) * L;
            const double sy = (double)((pc / 3) % 3 - 1) * L;
            const double sz = (double)(pc % 3 - 1) * L;
            v.x = (float)((px + sx - ox) * inv_len);
            v.y = (float)((py + sy - oy) * inv_len);
            v.z = (float)((pz + sz - oz) * inv_len);
            v.w = equal ? P.cut2 : pm;
            if (LOCAL) {
#pragma unroll
                for (int g = 0; g < GROUPS; ++g) {
                    const float4 c = qb[2 * g], h = qb[2 * g + 1];
                    const float gx = fmaxf(fabsf(v.x - c.x) - c.w, 0.f);
                    const float gy = fmaxf(fabsf(v.y - c.y) - h.x, 0.f);
                    const float gz = fmaxf(fabsf(v.z - c.z) - h.y, 0.f);
                    keep = keep || fmaf(gx, gx, fmaf(gy, gy, gz * gz)) < keep2;
                }
            } else {
                const float gx = fmaxf(fabsf(v.x) - hx, 0.f);
                const float gy = fmaxf(fabsf(v.y) - hy, 0.f);
                const float gz = fmaxf(fabsf(v.z) - hz, 0.f);
                keep = fmaf(gx, gx, fmaf(gy, gy, gz * gz)) < keep2;
            }
            if (!LOCAL) {
                v.x = (float)((px + sx) * inv_len);
                v.y = (float)((py + sy) * inv_len);
                v.z = (float)((pz + sz) * inv_len);
            }
        }
        const uint64_t bal = __ballot(keep);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        if (keep) tile[PACK ? count + rank + (count + rank) / kBlock : count + rank] = v;
        const int got = __popcll(bal);
        count += got;
        staged += got;
        // the next window's loads stay in flight while this tile is swept
        if (base + K * kBlock < s1) fetch(base + K * kBlock);
        if (count >= full) {
            wave_sync();
            float tx = 0.f, ty = 0.f, tz = 0.f;
            if (KAHAN) {
                if (equal) {
#pragma unroll 8
                    for (int q = 0; q < kBlock; ++q)
                        pair_f32_eq<NEWTON, TABLE>(tl[q], xi, yi, zi, tx, ty, tz, P.eps2n, tab);
                } else {
#pragma unroll 8
                    for (int q = 0; q < kBlock; ++q) pair_f32<NEWTON, TABLE>(tl[q], xi, yi, zi, P, tx, ty, tz, tab);
                }
                add_tiles(1 << lcopies, tx, ty, tz);
            } else {
#pragma unroll 8
                for (int q = 0; q < kBlock; ++q) pair_f32<NEWTON, TABLE>(tile[q], xi, yi, zi, P, ax, ay, az, tab);
            }
            wave_sync();
            count -= full;
            if (lane < count) tile[lane] = tile[PACK ? full + (full / kBlock) + lane : kBlock + lane];
            wave_sync();
        }
    }
    if (PACK && count > 0) {
        // the last tiles: the copies past them hold nothing
        wave_sync();
        float tx = 0.f, ty = 0.f, tz = 0.f;
        const int left = count - (lane >> (6 - lcopies)) * kBlock;     // entries from this copy's tile on
        const int most = count < kBlock ? count : kBlock;
        if (equal) {
#pragma unroll 1
            for (int q = 0; q < most; ++q)
                if (q < left) pair_f32_eq<NEWTON, TABLE>(tl[q], xi, yi, zi, tx, ty, tz, P.eps2n, tab);
        } else {
#pragma unroll 1
            for (int q = 0; q < most; ++q)
                if (q < left) pair_f32<NEWTON, TABLE>(tl[q], xi, yi, zi, P, tx, ty, tz, tab);
        }
        add_tiles((count + kBlock - 1) / kBlock, tx, ty, tz);
    }
    if (!PACK && count > 0) {
        wave_sync();
        float tx = 0.f, ty = 0.f, tz = 0.f;
        if (KAHAN) {
            if (equal) {
#pragma unroll 1
                for (int q = 0; q < count; ++q) pair_f32_eq<NEWTON, TABLE>(tile[q], xi, yi, zi, tx, ty, tz, P.eps2n, tab);
            } else {
#pragma unroll 1
                for (int q = 0; q < count; ++q) pair_f32<NEWTON, TABLE>(tile[q], xi, yi, zi, P, tx, ty, tz, tab);
            }
            kahan_add(ax, cx, tx);
            kahan_add(ay, cy, ty);
            kahan_add(az, cz, tz);
        } else {
#pragma unroll 1
            for (int q = 0; q < count; ++q) pair_f32<NEWTON, TABLE>(tile[q], xi, yi, zi, P, ax, ay, az, tab);
        }
    }
    // the sources this wave swept, for the statistics (summed when they are
    // asked for: an atomic per item on one counter costs 12 ns each, in turn)
    if (icount && lane == 0) icount[item * K + wv] = staged;
    // the compensated sums, then (K > 1) the waves' sums in wave order
    double sx = (double)ax - (double)cx, sy = (double)ay - (double)cy, sz = (double)az - (double)cz;
    if (K > 1) {
        __syncthreads();                 // every wave is done with the previous item's sums
        red[(wv * 3 + 0) * kBlock + lane] = sx;
        red[(wv * 3 + 1) * kBlock + lane] = sy;
        red[(wv * 3 + 2) * kBlock + lane] = sz;
        __syncthreads();
        if (wv != 0) return;
        sx = red[0 * kBlock + lane];
        sy = red[1 * kBlock + lane];
        sz = red[2 * kBlock + lane];
#pragma unroll
        for (int k = 1; k < K; ++k) {
            sx += red[(k * 3 + 0) * kBlock + lane];
            sy += red[(k * 3 + 1) * kBlock + lane];
            sz += red[(k * 3 + 2) * kBlock + lane];
        }
    }
    if (ia.acc && ia.ioff[b + 1] - ia.ioff[b] == 1) {
        // the block's only item: finish here, with the reduction's arithmetic
        const int64_t to = PACK ? (int64_t)ia.bstart[b] + tlane : t;
        if (PACK ? mine : lane < nt && target_on(ia, ia.perm[t])) {
            const int64_t i = ia.perm[to];
            const double sc = X.scale * (double)mu;
            put_acc(ia.acc, ia.wide, N, i, (float)(sx * sc), (float)(sy * sc), (float)(sz * sc));
        }
        return;
    }
    // the compensated sum (times the equal mass, if any), rounded once
    float* o = partial + item * 3 * kBlock;
    if (PACK && !mine) return;             // the reduction writes the active targets only
    o[0 * kBlock + tlane] = (float)(sx * (double)mu);
    o[1 * kBlock + tlane] = (float)(sy * (double)mu);
    o[2 * kBlock + tlane] = (float)(sz * (double)mu);
}

// Place of the r-th set bit of m (r below the number of set bits).
__device__ __forceinline__ int set_bit(uint64_t m, int r) {
    int at = 0;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        const int c = __popcll(m & ((1ull << d) - 1ull));
        if (r >= c) {
            r -= c;
            m >>= d;
            at += d;
        }
    }
    return at;
}

// Monopoles (sec. 3.3, 1 to N): one wave per target block walks the block's
// entries of the list expansion in order.  An entry contributes the node it
// stands for when the breadth-first expansion accepted it, and the leaves and
// groups of 8 leaves the depth-first walk accepted under it.  Each accepted
// node becomes a source of its mass at its centre of mass (FP64 sums,
// shifted by its periodic image, relative to the FP64 block centre, in units
// of ell), staged into an LDS ring like the particles of pp_item and swept
// with the same pair arithmetic and the same cut.  The result is added to
// the accelerations the PP path wrote.
// Bound by the pair arithmetic (8.0e9 pairs on 4 M clustered particles, 3.8 ms at
// the rate of pp_item).  One entry at a time, its few nodes in few lanes, took 9.7
// ms, bound by the latency of the loads; full waves of nodes take 5.6, and 4.8 with
// nodes beyond the cut dropped and the sweep unrolled.  Six waves per SIMD: 5.4.
__global__ void __launch_bounds__(64) monopole_kernel(ItemArgs ia, const FEntry* __restrict__ ent,
                                                      const int64_t* __restrict__ eoff,
                                                      const uint64_t* __restrict__ mono0,
                                                      const uint8_t* __restrict__ mono1,
                                                      const TreeView* __restrict__ tvs,
                                                      const double4* __restrict__ mc,
                                                      const double* __restrict__ pos_s, int64_t N,
                                                      int32_t* __restrict__ mcount) {
    __shared__ float4 tile[2 * kBlock];
    __shared__ uint64_t s_m0[kBlock];
    __shared__ int64_t s_first[kBlock];
    __shared__ int s_from[kBlock], s_m1[kBlock], s_sc[kBlock];
    const int64_t b = blockIdx.x;
    if (ia.sizes[kSkip] || b >= ia.sizes[kNBlock]) return;
    const int lane = threadIdx.x;
    if (mcount && lane == 0) mcount[b] = 0;
    if (ia.ioff[b + 1] == ia.ioff[b]) return;        // a block without active targets
    const int xbox = ia.bboxid[b];
    const BoxDev& X = ia.box[xbox];
    const TreeView& tv = tvs[xbox];
    const double L = X.L, cell = X.cell, inv_len = X.inv_len;
    PolyF32 P = X.poly;
    asm("" : "+v"(P.eps2n));                         // in VGPRs, as in pp_item
    asm("" : "+v"(P.cut2));
    const float keep2 = P.keep2;
    const IBox B = ia.bbox[b];
    const double ox = 0.5 * (double)(B.lo[0] + B.hi[0]) * cell;
    const double oy = 0.5 * (double)(B.lo[1] + B.hi[1]) * cell;
    const double oz = 0.5 * (double)(B.lo[2] + B.hi[2]) * cell;
    const float hx = (float)(0.5 * (double)(B.hi[0] - B.lo[0]) * cell * inv_len) * 1.0001f + 1e-6f;
    const float hy = (float)(0.5 * (double)(B.hi[1] - B.lo[1]) * cell * inv_len) * 1.0001f + 1e-6f;
    const float hz = (float)(0.5 * (double)(B.hi[2] - B.lo[2]) * cell * inv_len) * 1.0001f + 1e-6f;
    const int32_t nt = ia.bcount[b];
    const int64_t t = (int64_t)ia.bstart[b] + lane;
    float xi = 0.f, yi = 0.f, zi = 0.f;
    if (lane < nt) {
        xi = (float)((pos_s[t] - ox) * inv_len);
        yi = (float)((pos_s[N + t] - oy) * inv_len);
        zi = (float)((pos_s[2 * N + t] - oz) * inv_len);
    }
    float ax = 0.f, ay = 0.f, az = 0.f, cx = 0.f, cy = 0.f, cz = 0.f;
    int count = 0;
    int32_t taken = 0;
    // stage this lane's node (level, index) under shift code sc if `on`
    auto stage = [&](bool on, int lev, int64_t node, int sc) {
        bool some = false, keep = false;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (on) {
            const double4 m = mc[tv.off[lev] + node];
            if (m.w > 0.0) {
                some = true;
                const double sx = (double)(sc / 9 - 1) * L;
                const double sy = (double)((sc / 3) % 3 - 1) * L;
                const double sz = (double)(sc % 3 - 1) * L;
                v.x = (float)((m.x / m.w + sx - ox) * inv_len);
                v.y = (float)((m.y / m.w + sy - oy) * inv_len);
                v.z = (float)((m.z / m.w + sz - oz) * inv_len);
                v.w = (float)m.w;
                // a centre of mass beyond the cut of the block's box adds nothing
                const float gx = fmaxf(fabsf(v.x) - hx, 0.f);
                const float gy = fmaxf(fabsf(v.y) - hy, 0.f);
                const float gz = fmaxf(fabsf(v.z) - hz, 0.f);
                keep = fmaf(gx, gx, fmaf(gy, gy, gz * gz)) < keep2;
            }
        }
        const uint64_t bal = __ballot(keep);
        const int rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        if (keep) tile[count + rank] = v;
        count += __popcll(bal);
        taken += __popcll(__ballot(some));
        if (count >= kBlock) {
            wave_sync();
            float tx = 0.f, ty = 0.f, tz = 0.f;
#pragma unroll 8
            for (int q = 0; q < kBlock; ++q) pair_f32<false>(tile[q], xi, yi, zi, P, tx, ty, tz);
            kahan_add(ax, cx, tx);
            kahan_add(ay, cy, ty);
            kahan_add(az, cz, tz);
            wave_sync();
            count -= kBlock;
            if (lane < count) tile[lane] = tile[kBlock + lane];
            wave_sync();
        }
    };
    const int64_t e_end = eoff[b + 1];
    // nodes the breadth-first expansion accepted: one per entry, 64 entries
    // at a time
    for (int64_t e0 = eoff[b]; e0 < e_end; e0 += kBlock) {
        const int64_t e = e0 + lane;
        FEntry E{};
        const bool in = e < e_end;
        if (in) E = ent[e];
        stage(in && E.mono, E.lev, E.node, E.sc);
    }
    // leaves and groups of 8 leaves the depth-first walk accepted: 64 entries
    // at a time, their nodes numbered by a running count and taken 64 at a time
    if (mono0) {
        for (int64_t e0 = eoff[b]; e0 < e_end; e0 += kBlock) {
            const int64_t e = e0 + lane;
            const uint64_t m0 = e < e_end ? mono0[e] : 0ull;
            const uint32_t m1 = e < e_end ? mono1[e] : 0u;
            const int c = __popcll(m0) + __popc(m1);
            if (__ballot(c > 0) == 0ull) continue;
            int upto = c;
#pragma unroll
            for (int d = 1; d < kBlock; d <<= 1) {
                const int below = __shfl_up(upto, d);
                if (lane >= d) upto += below;
            }
            const int total = __builtin_amdgcn_readlane(upto, kBlock - 1);
            wave_sync();
            s_from[lane] = upto - c;
            s_m0[lane] = m0;
            s_m1[lane] = m1;
            if (c > 0) {
                const FEntry E = ent[e];
                s_first[lane] = (int64_t)E.node << (3 * E.lev);
                s_sc[lane] = E.sc;
            }
            wave_sync();
            for (int q0 = 0; q0 < total; q0 += kBlock) {
                const int q = q0 + lane;
                // the last entry that starts at or below q: the one that holds it
                int k = 0;
#pragma unroll
                for (int d = kBlock / 2; d > 0; d >>= 1)
                    if (s_from[k + d] <= q) k += d;
                int r = q - s_from[k];
                const uint64_t w0 = s_m0[k];
                const int c0 = __popcll(w0);
                const bool leaf = r < c0;
                const int64_t first = s_first[k];
                const int at = set_bit(leaf ? w0 : (uint64_t)s_m1[k], leaf ? r : r - c0);
                stage(q < total, leaf ? 0 : 1, (leaf ? first : first >> 3) + at, s_sc[k]);
            }
        }
    }
    if (count > 0) {
        wave_sync();
        float tx = 0.f, ty = 0.f, tz = 0.f;
        for (int q = 0; q < count; ++q) pair_f32<false>(tile[q], xi, yi, zi, P, tx, ty, tz);
        kahan_add(ax, cx, tx);
        kahan_add(ay, cy, ty);
        kahan_add(az, cz, tz);
    }
    if (taken == 0) return;
    if (lane < nt && target_on(ia, ia.perm[t])) {
        const int64_t i = ia.perm[t];
        const int64_t at = ia.wide ? 4 * i : i, row = ia.wide ? 1 : N;
        const float x = ia.acc[at], y = ia.acc[at + row], z = ia.acc[at + 2 * row];
        put_acc(ia.acc, ia.wide, N, i, x + (float)(((double)ax - (double)cx) * X.scale),
                y + (float)(((double)ay - (double)cy) * X.scale), z + (float)(((double)az - (double)cz) * X.scale));
    }
    if (mcount && lane == 0) mcount[b] = taken;
}

// One workgroup per item.
// Both forms are bounded to 6 waves per SIMD (80 VGPRs) with one wave per
// block and to 5 with more: two waves' VALU instructions can issue in the
// same cycle, so more resident waves keep the pair loop's issue slots
// fuller.
template <int VAR, int K>
__global__ void __launch_bounds__(64 * K, K > 1 ? 5 : 6) pp_f32_kernel(ItemArgs ia, const double* __restrict__ pos_s,
                                                        const float* __restrict__ mass_s, int64_t N,
                                                        float* __restrict__ partial,
                                                        int32_t* __restrict__ icount) {
    __shared__ float4 tile[K * tile_entries<VAR>()];
    __shared__ float4 qb[K * 8];
    __shared__ double red[K > 1 ? K * 3 * kBlock : 1];
    __shared__ float4 tab[(VAR & 8) ? kTabN : 1];
    __shared__ int mark[K * kBlock];
    if (ia.sizes[kSkip]) return;
    const int64_t nitem = ia.sizes[kNItem];
    const int64_t item = xcd_item(blockIdx.x, nitem);
    if (item < 0) return;
    if (VAR & 8) {
        for (int k = threadIdx.x; k < kTabN; k += 64 * K) tab[k] = ia.split_tab[k];
        __syncthreads();
    }
    pp_item<VAR, K>(ia, item, pos_s, mass_s, N, partial, icount, tile, tab, qb, red, mark);
}

// The same for launches of at most two waves per SIMD (short item lists,
// small boxes): compiled for two resident waves, so the register budget
// lets the compiler keep more of the unrolled sweep's pairs in flight, which
// a SIMD with only two waves to issue from needs.  Same arithmetic in the
// same order, so the same results.
template <int VAR, int K>
__global__ void __launch_bounds__(64 * K, 2) pp_f32_kernel_few(ItemArgs ia, const double* __restrict__ pos_s,
                                                               const float* __restrict__ mass_s, int64_t N,
                                                               float* __restrict__ partial,
                                                               int32_t* __restrict__ icount) {
    __shared__ float4 tile[K * tile_entries<VAR>()];
    __shared__ float4 qb[K * 8];
    __shared__ double red[K > 1 ? K * 3 * kBlock : 1];
    __shared__ float4 tab[(VAR & 8) ? kTabN : 1];
    __shared__ int mark[K * kBlock];
    if (ia.sizes[kSkip]) return;
    const int64_t nitem = ia.sizes[kNItem];
    const int64_t item = xcd_item(blockIdx.x, nitem);
    if (item < 0) return;
    if (VAR & 8) {
        for (int k = threadIdx.x; k < kTabN; k += 64 * K) tab[k] = ia.split_tab[k];
        __syncthreads();
    }
    pp_item<VAR, K>(ia, item, pos_s, mass_s, N, partial, icount, tile, tab, qb, red, mark);
}

// Persistent form: a fixed grid of waves pulls items from 8 queues (one
// contiguous stretch of items per XCD, as above); a wave first drains the
// queue of its own XCD, then steals from the others.  Every wave leaves
// once all queues are empty.  The item count is read from device memory,
// so the launch can be replayed from a graph while the lists change.
//
// Pops on one counter take about 12 ns each, in turn.  5120 waves that each
// popped all 8 queues once to find them empty spent about 60 us at the end of
// every launch, so a wave whose own queue ran dry reads the 8 counters with
// one load and pops only from queues that still hold items.
template <int VAR, int K>
__global__ void __launch_bounds__(64 * K, K > 1 ? 5 : 6) pp_f32_persistent(ItemArgs ia,
                                                            const double* __restrict__ pos_s,
                                                            const float* __restrict__ mass_s, int64_t N,
                                                            float* __restrict__ partial,
                                                            int32_t* __restrict__ icount,
                                                            unsigned* __restrict__ queues) {
    __shared__ float4 tile[K * tile_entries<VAR>()];
    __shared__ float4 qb[K * 8];
    __shared__ double red[K > 1 ? K * 3 * kBlock : 1];
    __shared__ float4 tab[(VAR & 8) ? kTabN : 1];
    __shared__ int mark[K * kBlock];
    __shared__ unsigned next_item;
    if (ia.sizes[kSkip]) return;
    if (VAR & 8) {
        for (int k = threadIdx.x; k < kTabN; k += 64 * K) tab[k] = ia.split_tab[k];
        __syncthreads();
    }
    const int64_t nitem = ia.sizes[kNItem];
    const int64_t per = (nitem + 7) / 8;
    const int my = blockIdx.x & 7;
    unsigned todo = 0xffu;               // bit v: queue (my + v) & 7 may hold items
    for (int v = 0; v < 8; ++v) {
        if (!(todo >> v & 1u)) continue;
        const int q = (my + v) & 7;
        const int64_t qbeg = q * per;
        const int64_t qend = qbeg + per < nitem ? qbeg + per : nitem;
        const unsigned qlen = qend > qbeg ? (unsigned)(qend - qbeg) : 0u;
        for (;;) {
            unsigned i = 0;
            if (K == 1) {
                if (threadIdx.x == 0) i = atomicAdd(&queues[q * kQueueStride], 1u);
                i = (unsigned)__builtin_amdgcn_readfirstlane((int)i);
            } else {
                // one pop per workgroup, shared through LDS
                __syncthreads();
                if (threadIdx.x == 0) next_item = atomicAdd(&queues[q * kQueueStride], 1u);
                __syncthreads();
                i = next_item;
            }
            if (i >= qlen) break;
            pp_item<VAR, K>(ia, qbeg + (int64_t)i, pos_s, mass_s, N, partial, icount, tile, tab, qb, red, mark);
        }
        if (v == 0) {
            // the other queues that still hold items (read by every wave: the
            // waves of a workgroup may differ, so the first one's word counts)
            const int w = threadIdx.x & 7;
            const int64_t left = nitem - ((my + w) & 7) * per;
            const unsigned head = __hip_atomic_load(&queues[((my + w) & 7) * kQueueStride], __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
            todo = (unsigned)__ballot((int64_t)head < (left < per ? left : per)) & 0xffu;
            if (K > 1) {
                __syncthreads();
                if (threadIdx.x == 0) next_item = todo;
                __syncthreads();
                todo = next_item;
            }
        }
    }
}

// Clears the work queues.
__global__ void reset_queues_kernel(unsigned* q) {
    if (threadIdx.x < 8) q[threadIdx.x * kQueueStride] = 0u;
}

// Sums of the items' staged sources: out[0] times the block's targets (the
// active ones where only they are swept), out[1] the lane slots of the sweeps
// (64 per staged source; with packed copies, of as many tiles at once, and of
// the fullest of the last tiles); with mcount, out[2]: the blocks' monopoles times
// their targets.  (out is cleared by the caller, and stays so after a pass whose
// kernels returned at once: they counted nothing.)
__global__ void __launch_bounds__(256) sum_staged_kernel(ItemArgs ia, const int32_t* __restrict__ icount,
                                                         int K, int packed,
                                                         const int32_t* __restrict__ mcount,
                                                         unsigned long long* __restrict__ out) {
    if (ia.sizes[kSkip]) return;
    unsigned long long ev = 0, ln = 0, mo = 0;
    if (mcount)
        for (int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; b < ia.sizes[kNBlock];
             b += (int64_t)gridDim.x * blockDim.x)
            mo += (unsigned long long)mcount[b] * (unsigned long long)ia.bcount[b];
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < ia.sizes[kNItem];
         it += (int64_t)gridDim.x * blockDim.x) {
        const int32_t b = ia.iblock[it];
        int targets = ia.bcount[b], lcopies = 0;
        if (packed) {
            const int na = __popcll(ia.bact[b]);
            lcopies = pack_copies(na);
            if (lcopies > 0) targets = na;
        }
        const unsigned full = (unsigned)kBlock << lcopies;
        for (int k = 0; k < K; ++k) {
            const unsigned c = (unsigned)icount[it * K + k], rest = c % full;
            ev += (unsigned long long)c * (unsigned long long)targets;
            ln += (unsigned long long)(c / full * kBlock + (rest < kBlock ? rest : kBlock)) * (unsigned long long)kBlock;
        }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        ev += __shfl_xor(ev, d);
        ln += __shfl_xor(ln, d);
        mo += __shfl_xor(mo, d);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(out, ev);
        atomicAdd(out + 1, ln);
        if (mcount) atomicAdd(out + 2, mo);
    }
}

__global__ void zero_u64_kernel(unsigned long long* p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

// One thread per (block, lane), grid-stride: sum the item partials of the
// block in order (FP64), scale by G / ell^2, scatter to input order.
__global__ void __launch_bounds__(256) reduce_f32_kernel(ItemArgs ia,
                                                         const float* __restrict__ partial,
                                                         const int32_t* __restrict__ perm,
                                                         int64_t N, float* __restrict__ acc) {
    if (ia.sizes[kSkip]) return;
    const int64_t nblock = ia.sizes[kNBlock];
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < nblock * kBlock;
         g += (int64_t)gridDim.x * blockDim.x) {
        const int64_t b = g / kBlock;
        const int l = (int)(g % kBlock);
        if (l >= ia.bcount[b]) continue;
        if (ia.ioff[b + 1] - ia.ioff[b] <= 1) continue;     // written by the PP kernel, or skipped
        double sx = 0, sy = 0, sz = 0;
        const int64_t end = ia.ioff[b + 1];
        int64_t it = ia.ioff[b];
        // four items' loads in flight at once; the sums keep item order
        for (; it + 4 <= end; it += 4) {
            float v[4][3];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const float* o = partial + (it + u) * 3 * kBlock;
                v[u][0] = o[0 * kBlock + l];
                v[u][1] = o[1 * kBlock + l];
                v[u][2] = o[2 * kBlock + l];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                sx += (double)v[u][0];
                sy += (double)v[u][1];
                sz += (double)v[u][2];
            }
        }
        for (; it < end; ++it) {
            const float* o = partial + it * 3 * kBlock;
            sx += (double)o[0 * kBlock + l];
            sy += (double)o[1 * kBlock + l];
            sz += (double)o[2 * kBlock + l];
        }
        const double scale = ia.box[ia.bboxid[b]].scale;
        const int64_t i = perm[(int64_t)ia.bstart[b] + l];
        if (!target_on(ia, i)) continue;
        put_acc(acc, ia.wide, N, i, (float)(sx * scale), (float)(sy * scale), (float)(sz * scale));
    }
}

// The records of put_acc to the caller's rows, active particles only.
__global__ void __launch_bounds__(256) unpack_acc_kernel(const float4* __restrict__ rec, int64_t N,
                                                         const int64_t* __restrict__ sizes,
                                                         const uint8_t* __restrict__ active,
                                                         float* __restrict__ acc) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (sizes[kSkip] || i >= N || (active && !active[i])) return;
    const float4 a = rec[i];
    acc[i] = a.x;
    acc[N + i] = a.y;
    acc[2 * N + i] = a.z;
}

// ------------------------------------------------------------------ FP64 --
// Per-box constants of the FP64 pair arithmetic.
struct F64Const {
    double eps2, rcut2;
    double tx;       // t of split_poly64.h per unit of s_eps
    double tz;       // log2(e) x^2 per unit of s_eps^2
};

// a b + c with c in scalar registers: written out because the compiler takes
// the two-operand form, with a copy of c into vector registers before every
// one (112 instructions per pair instead of 80).
__device__ __forceinline__ double fma_const(double a, double b, double c) {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(c));
    return r;
}

// One source at separation (dx, dy, dz), G m = gm, added into (tx, ty, tz).
// The separation and s^2 take the oracle's operation order (no contraction),
// so the cut decides as its own test does.  With y = 1 / s_eps from the
// hardware estimate and one third-order step, x = s_eps / 2 r_s and the split
// factor g = 2^-n 2^-f P(x) (split_poly64.h), the pair factor G m g y^3 holds
// about 4.7e-16 (relative, rms over the cut sphere, against 40 digits), and
// 5.5e-16 with the library's erfc, exp, square root and quotients.
__device__ __forceinline__ void pair_f64(double dx, double dy, double dz, double gm, const F64Const& C,
                                         double& tx, double& ty, double& tz) {
#pragma clang fp contract(off)
    const double s2 = dx * dx + dy * dy + dz * dz;
    const bool in = s2 < C.rcut2 && s2 > 0.0;
    const double se2 = s2 + C.eps2;
    const double y0 = __builtin_amdgcn_rsq(se2);
    const double e = fma(-(se2 * y0), y0, 1.0);
    const double y = fma(y0 * e, fma(e, 0.375, 0.5), y0);
    const double t = fma(se2 * y, C.tx, -1.0);
    double p = SPLIT64_P[SPLIT64_DEGREE_P];
#pragma unroll
    for (int j = SPLIT64_DEGREE_P - 1; j >= 0; --j) p = fma_const(p, t, SPLIT64_P[j]);
    const double z = se2 * C.tz;
    const double n = rint(z);
    const double f = z - n;
    double q = SPLIT64_E[SPLIT64_DEGREE_E];
#pragma unroll
    for (int j = SPLIT64_DEGREE_E - 1; j >= 0; --j) q = fma_const(q, f, SPLIT64_E[j]);
    q = ldexp(q, -(int)n);
    double F = ((y * y) * y) * ((q * p) * gm);
    F = in ? F : 0.0;
    tx = fma(F, dx, tx);
    ty = fma(F, dy, ty);
    tz = fma(F, dz, tz);
}

// FP64 sums (or, COUNT, the number of sources with s < r_cut, j != i) of one
// work item per wave: sources fetched, pruned against the four boxes of the
// block's runs of 16 targets (the FP32 kernel's test, which keeps too much
// only) and compacted into an LDS ring as in pp_item, then swept 64 at a time
// by all lanes.  The bound is FP64 issue: about 75 instructions per lane-pair
// at 4 clocks each.  The earlier form, library functions on every listed
// source with a branch per pair, held all of them (both branches of erfc
// among them) for one lane inside the cut: 262 k particles took 10.9 ms per
// call, now 3.4.
template <bool COUNT>
__global__ void __launch_bounds__(64) pp_f64_kernel(ItemArgs ia, const double* __restrict__ pos_s,
                                                    const double* __restrict__ mass_s, int64_t N,
                                                    double* __restrict__ partial,
                                                    int32_t* __restrict__ pcount) {
    if (ia.sizes[kSkip]) return;
    const int64_t nitem = ia.sizes[kNItem];
    const int64_t item = xcd_item(blockIdx.x, nitem);
    if (item < 0) return;
    constexpr int GROUPS = 4, GW = kBlock / GROUPS;
    __shared__ double4 tile[2 * kBlock];
    __shared__ double shift[2 * kBlock][3];
    __shared__ int32_t tj[COUNT ? 2 * kBlock : 1];
    __shared__ float4 qb[2 * GROUPS];
    __shared__ int mark[kBlock];
    const int lane = threadIdx.x;
    const int32_t b = ia.iblock[item];
    const int32_t s0 = ia.is0[item];
    const int32_t s1 = ia.is1[item];
    const int32_t nt = ia.bcount[b];
    const BoxDev& X = ia.box[ia.bboxid[b]];
    const double L = X.L, cell = X.cell, inv_len = X.inv_len, G = X.G;
    const float keep2 = fmaxf(X.poly.keep2, 1e-30f);     // a split scale far above the cut underflows its square
    F64Const C;
    C.eps2 = X.eps * X.eps;
    C.rcut2 = X.rcut * X.rcut;
    C.tx = 2.0 / SPLIT64_X_MAX / (2.0 * X.rs);
    C.tz = 1.4426950408889634 / (4.0 * X.rs * X.rs);
    const IBox B = ia.bbox[b];
    const double ox = 0.5 * (double)(B.lo[0] + B.hi[0]) * cell;
    const double oy = 0.5 * (double)(B.lo[1] + B.hi[1]) * cell;
    const double oz = 0.5 * (double)(B.lo[2] + B.hi[2]) * cell;
    const int64_t t = (int64_t)ia.bstart[b] + (lane < nt ? lane : 0);
    const double xi = pos_s[t], yi = pos_s[N + t], zi = pos_s[2 * N + t];
    {
        // boxes around the runs of 16 targets (lanes past the last target
        // repeat the first one), relative to the block centre in units of ell.
        // A half side is widened by the FP32 rounding of what the test
        // subtracts, too: at most 5 roundings of 2^-24 of the targets' offsets
        // (those of the cut itself are in keep2).  Offsets are large against
        // the cut where a grid cell is (few key bits)
        const float fx = (float)((xi - ox) * inv_len), fy = (float)((yi - oy) * inv_len),
                    fz = (float)((zi - oz) * inv_len);
        float ax_ = fx, bx_ = fx, ay_ = fy, by_ = fy, az_ = fz, bz_ = fz;
#pragma unroll
        for (int m = 1; m < GW; m <<= 1) {
            ax_ = fminf(ax_, __shfl_xor(ax_, m));
            bx_ = fmaxf(bx_, __shfl_xor(bx_, m));
            ay_ = fminf(ay_, __shfl_xor(ay_, m));
            by_ = fmaxf(by_, __shfl_xor(by_, m));
            az_ = fminf(az_, __shfl_xor(az_, m));
            bz_ = fmaxf(bz_, __shfl_xor(bz_, m));
        }
        if (lane % GW == 0) {
            const int g = lane / GW;
            auto half = [](float a, float b) {
                return 0.5f * (b - a) * 1.0001f + 1e-6f + 5e-7f * fmaxf(fabsf(a), fabsf(b));
            };
            qb[2 * g] = make_float4(0.5f * (ax_ + bx_), 0.5f * (ay_ + by_), 0.5f * (az_ + bz_), half(ax_, bx_));
            qb[2 * g + 1] = make_float4(half(ay_, by_), half(az_, bz_), 0.f, 0.f);
        }
        wave_sync();
    }
    const int64_t r_lo = ia.roff[b], r_hi = ia.roff[b + 1] - 1;
    int64_t rcur = s1 > s0 ? find_range_wave(ia.rpre, r_lo, r_hi, s0) : r_lo;
    double ax = 0, ay = 0, az = 0;
    int32_t cnt = 0;
    int count = 0, shifted = 0;      // staged sources; the last shifted one's ring index + 1
    double px = 0, py = 0, pz = 0, pm = 0;
    int pc = 13;
    int32_t pj = -1;
    bool pv = false;
    auto fetch = [&](int32_t base) {
        const int32_t p = base + lane;
        pv = p < s1;
        int32_t rb, rp;
        int code;
        const int64_t r = window_range<1>(ia, base, s1, rcur, r_hi, mark, rb, rp, code);
        if (pv) {
            const int64_t j = (int64_t)rb + (p - rp);
            pc = code;
            pj = (int32_t)j;
            px = pos_s[j];
            py = pos_s[N + j];
            pz = pos_s[2 * N + j];
            if (!COUNT) pm = mass_s[j];
        }
        rcur = readlane64(r, kBlock - 1);
    };
    auto sweep = [&](int n) {
#pragma clang fp contract(off)
        double tx = 0, ty = 0, tz = 0;
        if (shifted > 0) {
            for (int q = 0; q < n; ++q) {
                const double4 s = tile[q];
                // (x_j - x_i), then the periodic shift: the order of the
                // minimum-image difference
                const double dx = (s.x - xi) + shift[q][0];
                const double dy = (s.y - yi) + shift[q][1];
                const double dz = (s.z - zi) + shift[q][2];
                if (COUNT) cnt += dx * dx + dy * dy + dz * dz < C.rcut2 && tj[q] != (int32_t)t ? 1 : 0;
                else pair_f64(dx, dy, dz, s.w, C, tx, ty, tz);
            }
        } else {
            for (int q = 0; q < n; ++q) {
                const double4 s = tile[q];
                const double dx = s.x - xi, dy = s.y - yi, dz = s.z - zi;
                if (COUNT) cnt += dx * dx + dy * dy + dz * dz < C.rcut2 && tj[q] != (int32_t)t ? 1 : 0;
                else pair_f64(dx, dy, dz, s.w, C, tx, ty, tz);
            }
        }
        ax += tx;
        ay += ty;
        az += tz;
    };
    if (s0 < s1) fetch(s0);
    for (int32_t base = s0; base < s1; base += kBlock) {
        bool keep = false;
        const double sx = (double)(pc / 9 - 1) * L;
        const double sy = (double)((pc / 3) % 3 - 1) * L;
        const double sz = (double)(pc % 3 - 1) * L;
        if (pv) {
            const float vx = (float)((px + sx - ox) * inv_len);
            const float vy = (float)((py + sy - oy) * inv_len);
            const float vz = (float)((pz + sz - oz) * inv_len);
#pragma unroll
            for (int g = 0; g < GROUPS; ++g) {
                const float4 c = qb[2 * g], h = qb[2 * g + 1];
                const float gx = fmaxf(fabsf(vx - c.x) - c.w, 0.f);
                const float gy = fmaxf(fabsf(vy - c.y) - h.x, 0.f);
                const float gz = fmaxf(fabsf(vz - c.z) - h.y, 0.f);
                keep = keep || fmaf(gx, gx, fmaf(gy, gy, gz * gz)) < keep2;
            }
        }
        const uint64_t bal = __ballot(keep), far = __ballot(keep && pc != 13);
        const int at = count + __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
        if (keep) {
            tile[at] = make_double4(px, py, pz, G * pm);
            shift[at][0] = sx;
            shift[at][1] = sy;
            shift[at][2] = sz;
            if (COUNT) tj[at] = pj;
        }
        count += __popcll(bal);
        if (far) shifted = count;
        if (base + kBlock < s1) fetch(base + kBlock);
        if (count >= kBlock) {
            wave_sync();
            sweep(kBlock);
            wave_sync();
            count -= kBlock;
            shifted -= kBlock;
            if (lane < count) {
                tile[lane] = tile[kBlock + lane];
                for (int k = 0; k < 3; ++k) shift[lane][k] = shift[kBlock + lane][k];
                if (COUNT) tj[lane] = tj[kBlock + lane];
            }
            wave_sync();
        }
    }
    if (count > 0) {
        wave_sync();
        sweep(count);
    }
    if (COUNT) {
        pcount[item * kBlock + lane] = cnt;
    } else {
        double* o = partial + item * 3 * kBlock;
        o[0 * kBlock + lane] = ax;
        o[1 * kBlock + lane] = ay;
        o[2 * kBlock + lane] = az;
    }
}

__global__ void __launch_bounds__(256) reduce_f64_kernel(ItemArgs ia,
                                                         const double* __restrict__ partial,
                                                         const int32_t* __restrict__ perm,
                                                         int64_t N, double* __restrict__ acc) {
    if (ia.sizes[kSkip]) return;
    const int64_t nblock = ia.sizes[kNBlock];
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t b = g / kBlock;
    const int l = (int)(g % kBlock);
    if (b >= nblock || l >= ia.bcount[b]) return;
    double sx = 0, sy = 0, sz = 0;
    for (int64_t it = ia.ioff[b]; it < ia.ioff[b + 1]; ++it) {
        const double* o = partial + it * 3 * kBlock;
        sx += o[0 * kBlock + l];
        sy += o[1 * kBlock + l];
        sz += o[2 * kBlock + l];
    }
    const int64_t i = perm[(int64_t)ia.bstart[b] + l];
    acc[i] = sx;
    acc[N + i] = sy;
    acc[2 * N + i] = sz;
}

__global__ void __launch_bounds__(256) reduce_count_kernel(ItemArgs ia,
                                                           const int32_t* __restrict__ pc,
                                                           const int32_t* __restrict__ perm,
                                                           int64_t* __restrict__ counts,
                                                           unsigned long long* __restrict__ total) {
    if (ia.sizes[kSkip]) return;
    const int64_t nblock = ia.sizes[kNBlock];
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t b = g / kBlock;
    const int l = (int)(g % kBlock);
    if (b >= nblock || l >= ia.bcount[b]) return;
    int64_t s = 0;
    for (int64_t it = ia.ioff[b]; it < ia.ioff[b + 1]; ++it) s += pc[it * kBlock + l];
    if (counts) counts[perm[(int64_t)ia.bstart[b] + l]] = s;
    atomicAdd(total, (unsigned long long)s);
}

}  // namespace

double pair_length_unit(const pp_box_params& p) {
    return 2.0 * p.rs * std::sqrt(0.5 * SPLIT_POLY_U_MAX);
}

int make_poly(const pp_box_params& p, PolyF32* out) {
    const double ell = pair_length_unit(p);
    double e2 = (p.eps / ell) * (p.eps / ell);
    const double floor2 = ldexp(1.0, -60);          // keeps y^3 finite for s = eps = 0
    if (e2 < floor2) e2 = floor2;
    const double c2 = (p.rcut / ell) * (p.rcut / ell);
    out->eps2n = (float)e2;
    out->cut2 = (float)(c2 + e2);
    out->keep2 = (float)c2 * 1.0002f;
    out->pad = 0.f;
    return PP_OK;
}

// H(u) = (1 - g(x)) / x^3, u = x^2, from g'(x) = -(4/sqrt(pi)) x^2 e^{-x^2}:
// 1 - g(x) = (4/sqrt(pi)) sum_n (-1)^n x^{2n+3} / (n! (2n+3)), so
// H(u) = (4/sqrt(pi)) sum_n (-u)^n / (n! (2n+3)).  In FP64 the alternating
// terms stay below 40 for u <= 5.2, so the sum keeps about 14 digits.
__device__ double split_H_series(double u) {
    double term = 1.0, sum = 1.0 / 3.0;
    for (int n = 1; n < 80; ++n) {
        term *= -u / (double)n;
        sum += term / (double)(2 * n + 3);
        if (fabs(term) < 1e-18) break;
    }
    return 4.0 / 1.7724538509055160272981674833411 * sum;
}

// Piece k of the table covers r2 in [2k/N, 2(k+1)/N); the quadratic through
// the piece's two ends and midpoint, in z = position inside the piece.
__global__ void split_table_kernel(float4* __restrict__ tab) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= kTabN) return;
    const double hu = 0.5 * SPLIT_POLY_U_MAX;           // u per unit of r2
    const double w = 2.0 / kTabN;
    const double f0 = kHScale * split_H_series(hu * (k * w));
    const double fm = kHScale * split_H_series(hu * ((k + 0.5) * w));
    const double f1 = kHScale * split_H_series(hu * ((k + 1) * w));
    tab[k] = make_float4((float)f0, (float)(-3.0 * f0 + 4.0 * fm - f1), (float)(2.0 * f0 - 4.0 * fm + 2.0 * f1),
                         0.f);
}

int launch_split_table(Work& w, hipStream_t s) {
    PP_TRY(w.split_tab.reserve(sizeof(float4) * kTabN));
    hipLaunchKernelGGL(split_table_kernel, dim3(1), dim3(kTabN), 0, s, w.split_tab.as<float4>());
    PP_HIP(hipGetLastError());
    return PP_OK;
}

// CUs of the current device.
static int cu_count(int* cus) {
    int dev = 0;
    *cus = 256;
    PP_HIP(hipGetDevice(&dev));
    PP_HIP(hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev));
    return PP_OK;
}

// Workgroups of the persistent launch: waves_per_cu waves per CU in
// workgroups of K waves.
static int64_t persistent_groups(int cus, int waves_per_cu, int K) {
    const int wpc = waves_per_cu > 0 ? waves_per_cu : 16;
    return (int64_t)cus * ((wpc + K - 1) / K);
}

// The persistent form is launched as one workgroup per item when the last
// call's items were short, or fit the chip in one go: the hardware's dispatch
// then hands them out faster than the queues, whose pops take 12 ns each, in
// turn.  300 k clustered particles (65 k items of 512 positions): 0.86 ms
// against 1.01 queued; 1 M uniform ones in items of 256: 1.37 against 1.65 ms,
// of 1024 (mean 916): 1.38 against 1.42.  Long items run as fast or faster
// queued (1.2 M at 2048 positions, mean 1600: 1.94 against 1.99 ms; 16.8 M:
// 342.6 against 344.6).  Both forms give the same results, so the last call's
// mean is only a hint; before the first call the room for items stands in.
constexpr int64_t kGridFew = 8192, kGridFirst = 65536;
constexpr int64_t kGridLength = 1000;

int f32_grid_groups(const Work& w, int waves_per_block, Mode mode, int64_t* groups) {
    const int64_t room = w.cap_item * waves_per_block;
    const bool grid = mode == Mode::kGrid || room <= kGridFew ||
                      (w.nitem > 0 ? w.total_src / w.nitem < kGridLength * waves_per_block : room <= kGridFirst);
    *groups = grid ? xcd_groups(w.cap_item) : 0;
    // a launch takes fewer than 2^32 threads; the queues take any number of items
    if (mode != Mode::kGrid && *groups * waves_per_block * kBlock > (int64_t)UINT32_MAX) *groups = 0;
    return PP_OK;
}

template <int VAR, int K>
static int launch_pp_f32_var(const ItemArgs& ia, const Work& w, Mode mode, int waves_per_cu,
                             float* partial, int32_t* icount, unsigned* queues, hipStream_t s) {
    if (w.cap_item == 0) return PP_OK;
    int cus = 256;
    int64_t grid = 0;
    PP_TRY(cu_count(&cus));
    PP_TRY(f32_grid_groups(w, K, mode, &grid));
    if (grid == 0) {
        const int64_t groups = persistent_groups(cus, waves_per_cu, K);
        hipLaunchKernelGGL(reset_queues_kernel, dim3(1), dim3(64), 0, s, queues);
        hipLaunchKernelGGL((pp_f32_persistent<VAR, K>), dim3((unsigned)groups), dim3(kBlock * K), 0, s, ia,
                           w.pos_s.as<double>(), w.mass_s.as<float>(), w.pos_n, partial, icount, queues);
    } else {
        // one workgroup per item, up to the item capacity (the count is on
        // the device; the workgroups past it return at once)
        // At most two waves per SIMD by the last call's item count (a hint
        // only: both forms give the same results), the form built for that.
        bool few = false;
        if constexpr ((VAR & 7) == 0) {
            few = w.nitem > 0 && w.nitem * K <= 2 * 4 * (int64_t)cus;
            if (few)
                hipLaunchKernelGGL((pp_f32_kernel_few<VAR, K>), dim3((unsigned)grid), dim3(kBlock * K), 0,
                                   s, ia, w.pos_s.as<double>(), w.mass_s.as<float>(), w.pos_n, partial, icount);
        }
        if (!few)
            hipLaunchKernelGGL((pp_f32_kernel<VAR, K>), dim3((unsigned)grid), dim3(kBlock * K), 0, s,
                               ia, w.pos_s.as<double>(), w.mass_s.as<float>(), w.pos_n, partial, icount);
    }
    PP_HIP(hipGetLastError());
    return PP_OK;
}

template <int K>
static int launch_pp_f32_k(const ItemArgs& ia, const Work& w, Mode mode, int waves_per_cu,
                           int variant, float* partial, int32_t* icount,
                           unsigned* queues, hipStream_t s) {
    switch (variant) {
        case 16: return launch_pp_f32_var<16, K>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 24: return launch_pp_f32_var<24, K>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 0: return launch_pp_f32_var<0, K>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 8: return launch_pp_f32_var<8, K>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        default: return fail(PP_EINVAL, "more than one wave per block needs variant 0 or 8");
    }
}

// Whether a launch over active targets packs them (pp_item, PACK).
static bool packs_active(const Work& w, int variant) { return w.active && (variant & 7) == 0; }

int launch_pp_f32(const BatchDev& bd, const Work& w, int waves_per_block, Mode mode, int waves_per_cu,
                  int variant, float* partial, float* acc, int32_t* icount,
                  unsigned* queues, hipStream_t s) {
    ItemArgs ia = item_args(bd, w);
    ia.acc = acc;
    variant &= 15;
    if (packs_active(w, variant)) variant |= 16;
    if (waves_per_block == 2)
        return launch_pp_f32_k<2>(ia, w, mode, waves_per_cu, variant, partial, icount, queues, s);
    if (waves_per_block == 4)
        return launch_pp_f32_k<4>(ia, w, mode, waves_per_cu, variant, partial, icount, queues, s);
    if (waves_per_block == 8)
        return launch_pp_f32_k<8>(ia, w, mode, waves_per_cu, variant, partial, icount, queues, s);
    switch (variant) {
        case 16: return launch_pp_f32_var<16, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 24: return launch_pp_f32_var<24, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 0: return launch_pp_f32_var<0, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 1: return launch_pp_f32_var<1, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 2: return launch_pp_f32_var<2, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 3: return launch_pp_f32_var<3, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 4: return launch_pp_f32_var<4, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 5: return launch_pp_f32_var<5, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 6: return launch_pp_f32_var<6, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 7: return launch_pp_f32_var<7, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 8: return launch_pp_f32_var<8, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 9: return launch_pp_f32_var<9, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 10: return launch_pp_f32_var<10, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 11: return launch_pp_f32_var<11, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 12: return launch_pp_f32_var<12, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 13: return launch_pp_f32_var<13, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        case 14: return launch_pp_f32_var<14, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
        default: return launch_pp_f32_var<15, 1>(ia, w, mode, waves_per_cu, partial, icount, queues, s);
    }
}

int launch_monopole(const BatchDev& bd, const Work& w, float* acc, int32_t* mcount, hipStream_t s) {
    if (w.cap_block == 0 || !w.ent_final) return PP_OK;
    ItemArgs ia = item_args(bd, w);
    ia.acc = acc;
    hipLaunchKernelGGL(monopole_kernel, dim3((unsigned)w.cap_block), dim3(kBlock), 0, s, ia, w.ent_final,
                       w.eoff.as<int64_t>(), w.mono0, w.mono1, w.tviews.as<TreeView>(),
                       w.tree_mc.as<double4>(), w.pos_s.as<double>(), w.pos_n, mcount);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int launch_sum_staged(const BatchDev& bd, const Work& w, int waves_per_block, int variant, const int32_t* icount,
                      const int32_t* mcount, unsigned long long* out, hipStream_t s) {
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, s, out, 3);
    hipLaunchKernelGGL(sum_staged_kernel, dim3(256), dim3(256), 0, s, item_args(bd, w), icount, waves_per_block,
                       packs_active(w, variant) ? 1 : 0, mcount, out);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int launch_unpack_acc(const Work& w, const float* rec, float* acc, hipStream_t s) {
    hipLaunchKernelGGL(unpack_acc_kernel, dim3(blocks_for(w.pos_n, 256)), dim3(256), 0, s,
                       reinterpret_cast<const float4*>(rec), w.pos_n, w.sizes.as<int64_t>(), w.active, acc);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int launch_reduce_f32(const BatchDev& bd, const Work& w, const float* partial, float* acc,
                      hipStream_t s) {
    ItemArgs ia = item_args(bd, w);
    // a fixed grid (grid-stride) so a captured graph stays valid as nblock changes
    hipLaunchKernelGGL(reduce_f32_kernel, dim3(2048), dim3(256), 0, s, ia, partial,
                       w.perm.as<int32_t>(), w.pos_n, acc);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int launch_pp_f64(const BatchDev& bd, const Work& w, double* partial, hipStream_t s) {
    if (w.cap_item == 0) return PP_OK;
    ItemArgs ia = item_args(bd, w);
    hipLaunchKernelGGL(pp_f64_kernel<false>, dim3((unsigned)xcd_groups(w.cap_item)), dim3(kBlock), 0, s, ia,
                       w.pos_s.as<double>(), w.mass_sd.as<double>(), w.pos_n, partial,
                       (int32_t*)nullptr);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int launch_reduce_f64(const BatchDev& bd, const Work& w, const double* partial, double* acc,
                      hipStream_t s) {
    if (w.cap_block == 0) return PP_OK;
    ItemArgs ia = item_args(bd, w);
    hipLaunchKernelGGL(reduce_f64_kernel, dim3(blocks_for(w.cap_block * kBlock, 256)), dim3(256), 0, s,
                       ia, partial, w.perm.as<int32_t>(), w.pos_n, acc);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int launch_count(const BatchDev& bd, const Work& w, int32_t* partial, hipStream_t s) {
    if (w.cap_item == 0) return PP_OK;
    ItemArgs ia = item_args(bd, w);
    hipLaunchKernelGGL(pp_f64_kernel<true>, dim3((unsigned)xcd_groups(w.cap_item)), dim3(kBlock), 0, s, ia,
                       w.pos_s.as<double>(), (const double*)nullptr, w.pos_n,
                       (double*)nullptr, partial);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int launch_reduce_count(const BatchDev& bd, const Work& w, const int32_t* partial, int64_t* counts,
                        unsigned long long* total, hipStream_t s) {
    if (w.cap_block == 0) return PP_OK;
    ItemArgs ia = item_args(bd, w);
    hipLaunchKernelGGL(reduce_count_kernel, dim3(blocks_for(w.cap_block * kBlock, 256)), dim3(256), 0,
                       s, ia, partial, w.perm.as<int32_t>(), counts, total);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

}  // namespace pp
