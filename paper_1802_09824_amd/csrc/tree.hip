// Octree leaves, the implicit trees over them, and the near-leaf lists, for
// a batch of boxes.
//
// Leaves (sec. 3.2-3.3): with particles in Peano-Hilbert key order every
// octree node (the particles sharing the top 3l key bits) is a contiguous
// run.  A leaf is a maximal node holding at most M = leaf_max particles
// ("a leaf is a package of a given number of particles", sec. 3.3).  The
// level of the leaf of particle k is found without building the tree: the
// level-l node of k holds more than M particles iff some run of M + 1
// consecutive particles (of the same box) containing k shares its top 3l
// key bits, so
//   level(k) = 1 + max over s in [k - M, k] of lcp(key[s], key[s + M])
// (lcp in 3-bit digits, capped at b; 0 when no such run exists).
//
// Near lists (sec. 3.3, the N-to-M leaf pairs of the dual tree traversal,
// restricted to the short range): an implicit 8-ary tree over each box's
// leaf array (leaves are in key order, so consecutive leaves are close in
// space) is walked, pruning subtrees whose integer bounding box is at least
// r_cut away.  The leaf test is exact integer arithmetic, identical for the
// canonical list and for the block lists.
#include <algorithm>
#include "lookback.h"

namespace pp {
namespace {

#pragma clang fp contract(off)
// Grid cell of one coordinate of an already wrapped position w (the gather
// stores x - L floor(x / L)): floor(w 2^b / L) clamped, exactly the
// quantisation the key kernel applies to the same wrapped value.
__device__ __forceinline__ uint32_t quantise_w(double w, double L, double scale, uint32_t qmax) {
    (void)L;
    double f = floor(w * scale);
    if (!(f > 0.0)) return 0u;
    if (f > (double)qmax) return qmax;
    return (uint32_t)f;
}
#pragma clang fp contract(on)

__device__ __forceinline__ int common_digits(uint64_t a, uint64_t b, int bits) {
    uint64_t x = a ^ b;
    if (x == 0) return bits;
    int lz = __clzll((long long)x);
    return (lz - (64 - 3 * bits)) / 3;
}

__device__ __forceinline__ uint64_t key_prefix(uint64_t key, int level, int bits) {
    return level == 0 ? 0ull : key >> (3 * (bits - level));
}

// The shape of one box's tree over c0 leaves: level h has cnt_h =
// ceil(cnt_{h-1} / 8) nodes while cnt_{h-1} > 1.
__device__ __forceinline__ int64_t level_count(int64_t c0, int h) {
    int64_t c = c0;
    for (int k = 0; k < h; ++k) {
        if (c <= 1) return 0;
        c = (c + 7) / 8;
    }
    return c;
}

// The level the list expansion starts from: the lowest one above the leaves
// with at most `most` nodes (the only level of a one-leaf tree).
__device__ __forceinline__ int start_level(int64_t c0, int64_t most) {
    int64_t c = c0;
    int h = 0;
    while (c > 1 && (h == 0 || c > most)) {
        c = (c + 7) / 8;
        ++h;
    }
    return h;
}

// Leaves per workgroup of the kernel that builds levels 0 to 3.
constexpr int kTreeGroup = 512;

// Tree view, per-level prefixes and group prefix of the only box of a batch
// of one (see tree_views_kernel, which does it for several boxes).
__device__ void one_tree_view(int64_t c0, int64_t start_nodes, TreeView* tv, int64_t* lp, int64_t* gp,
                              int64_t* sizes) {
    int64_t base = 0, c = c0;
    int nl = 0;
    for (int h = 0; h < kTreeMaxLevels; ++h) {
        tv->cnt[h] = c;
        tv->off[h] = c > 0 ? base : 0;
        lp[2 * h] = 0;
        lp[2 * h + 1] = c;
        if (c > 0) nl = h + 1;
        base += c;
        c = c <= 1 ? 0 : (c + 7) / 8;
    }
    tv->loff = 0;
    tv->nlev = nl;
    tv->start = start_level(c0, start_nodes);
    gp[0] = 0;
    gp[1] = (c0 + kTreeGroup - 1) / kTreeGroup;
    sizes[kStart] = tv->start;
}

// Leaves of a tile of 256 IPT consecutive particles (key order) of all boxes:
// lcp(key[s], key[s + M]) of the tile and the M particles before it goes to
// LDS, its sliding maximum over M + 1 entries by doubling gives the particles'
// leaf levels, a particle starts a leaf where its prefix at the level of the
// particle before it differs, and the leaf numbers come from a ballot count,
// the tile's running sums and the look-back over the earlier tiles.
// One launch in the place of seven (lcp, block maxima, levels, flags, scan,
// box offsets, fill): 59 us of kernels on 2.1 M particles became 41, and on
// 32 k the launches themselves were the cost.
template <int IPT>
__global__ void __launch_bounds__(256) leaves_kernel(BatchDev bd, const uint64_t* __restrict__ keys, int64_t N,
                                                     LbArgs lb, int64_t ntile, int64_t* __restrict__ begin,
                                                     int32_t* __restrict__ level,
                                                     uint64_t* __restrict__ prefix,
                                                     int64_t* __restrict__ loff, int64_t* __restrict__ sizes,
                                                     int64_t start_nodes, TreeView* __restrict__ tv,
                                                     int64_t* __restrict__ lp, int64_t* __restrict__ gp) {
    constexpr int TS = 256 * IPT;
    constexpr int LEN = TS + 1 + 1024;              // leaf_max is at most 1024
    __shared__ int8_t lam[2][LEN];
    __shared__ unsigned s_tile;
    __shared__ int s_seg[IPT * 4];
    __shared__ int64_t s_pre;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int M = bd.leaf_max, W = M + 1;
    lb_clear_other(lb);
    if (t == 0) s_tile = (unsigned)atomicAdd(lb.cur, 1ull);
    __syncthreads();
    const int64_t tile = s_tile;
    const int64_t t0 = tile * TS;
    // lam[.][i]: run of M + 1 particles that ends at particle t0 - 1 + i
    const int len = TS + 1 + M;
    for (int i = t; i < len; i += 256) {
        const int64_t e = t0 - 1 + i, s = e - M;
        int8_t v = -1;
        if (s >= 0 && e < N && (bd.nbox == 1 || bd.poff[box_of(bd.poff, bd.nbox, s) + 1] > e))
            v = (int8_t)common_digits(keys[s], keys[e], bd.bits);
        lam[0][i] = v;
    }
    __syncthreads();
    int cur = 0, span = 1;
    for (; 2 * span <= W; span *= 2) {
        for (int i = t; i < len; i += 256) {
            const int8_t a = lam[cur][i], b = i + span < len ? lam[cur][i + span] : (int8_t)-1;
            lam[cur ^ 1][i] = a > b ? a : b;
        }
        __syncthreads();
        cur ^= 1;
    }
    // level of particle t0 - 1 + i (0 <= i <= TS)
    auto level_at = [&](int i) {
        const int a = lam[cur][i], b = lam[cur][i + W - span];
        const int m = a > b ? a : b;
        return m < 0 ? 0 : (m + 1 < bd.bits ? m + 1 : bd.bits);
    };
    uint64_t starts[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const int i = j * 256 + t;
        const int64_t k = t0 + i;
        bool f = false;
        if (k < N) {
            f = true;
            if (k > 0 && (bd.nbox == 1 || bd.poff[box_of(bd.poff, bd.nbox, k)] < k)) {
                const int l = level_at(i);           // of the particle before
                f = key_prefix(keys[k], l, bd.bits) != key_prefix(keys[k - 1], l, bd.bits);
            }
        }
        starts[j] = __ballot(f);
        if (lane == 0) s_seg[j * 4 + wave] = __popcll(starts[j]);
    }
    __syncthreads();
    int64_t agg = 0;
    for (int k = 0; k < IPT * 4; ++k) agg += s_seg[k];
    if (wave == 0) {
        const int64_t ex = lb_tile_prefix<1>(lb, tile, 0, agg, sizes, lane);
        if (lane == 0) s_pre = ex;
    }
    __syncthreads();
    const int64_t pre = s_pre;
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        int64_t a = pre;
        for (int k = 0; k < j * 4 + wave; ++k) a += s_seg[k];
        a += __popcll(starts[j] & ((1ull << lane) - 1ull));
        const int i = j * 256 + t;
        const int64_t k = t0 + i;
        if (!(starts[j] >> lane & 1ull)) continue;
        const int l = level_at(i + 1);
        begin[a] = k;
        level[a] = l;
        prefix[a] = key_prefix(keys[k], l, bd.bits);
        // every box start starts a leaf, the first one of its box (and of the
        // empty boxes before it)
        int x = box_of(bd.poff, bd.nbox, k);
        if (bd.poff[x] == k) {
            loff[x] = a;
            for (; x > 0 && bd.poff[x - 1] == k; --x) loff[x - 1] = a;
        }
    }
    if (tile == ntile - 1 && t == 0) {
        const int64_t total = pre + agg;
        sizes[kNLeaf] = total;
        for (int x = bd.nbox; x >= 0 && bd.poff[x] == N; --x) loff[x] = total;
        if (bd.nbox == 1) one_tree_view(total, start_nodes, tv, lp, gp, sizes);
    }
}

// No particles: no leaves.
__global__ void no_leaves_kernel(int nbox, int64_t* __restrict__ loff, int64_t* __restrict__ sizes,
                                 int64_t start_nodes, TreeView* __restrict__ tv, int64_t* __restrict__ lp,
                                 int64_t* __restrict__ gp) {
    for (int x = threadIdx.x; x <= nbox; x += blockDim.x) loff[x] = 0;
    if (threadIdx.x != 0) return;
    sizes[kNLeaf] = 0;
    if (nbox == 1) one_tree_view(0, start_nodes, tv, lp, gp, sizes);
}

// Levels 0 to 3 of every box's tree, one workgroup per kTreeGroup leaves (a
// whole level-3 node): the leaves' counts and integer boxes from their
// particles, then the unions of up to 8 nodes, level by level, in LDS.
// Bound by the particles' loads (48 MB at 2.1 M: 9 us) and their latency; a
// launch for the leaves and one per level took 72 us there, these levels and
// the rest in tree_top_kernel take 47, and a small box two launches, not 6.
// gp: groups of the boxes before each box.
__global__ void __launch_bounds__(kTreeGroup) leaf_tree_kernel(BatchDev bd, const double* __restrict__ pos_s,
                                                               int64_t N, const TreeView* __restrict__ tvs,
                                                               const int64_t* __restrict__ gp,
                                                               const int64_t* __restrict__ begin,
                                                               const int64_t* __restrict__ sizes,
                                                               int32_t* __restrict__ count,
                                                               IBox* __restrict__ nodes) {
    __shared__ IBox s_box[kTreeGroup];
    const int64_t g = blockIdx.x;
    if (g >= gp[bd.nbox]) return;
    const int x = box_of(gp, bd.nbox, g);
    const TreeView& T = tvs[x];
    const BoxDev& X = bd.box[x];
    const int t = threadIdx.x;
    int64_t i = (g - gp[x]) * kTreeGroup + t;        // leaf of the box
    IBox B;
    for (int ax = 0; ax < 3; ++ax) {
        B.lo[ax] = INT32_MAX;
        B.hi[ax] = INT32_MIN;
    }
    if (i < T.cnt[0]) {
        const int64_t a = T.loff + i, m = sizes[kNLeaf];
        const int64_t b0 = begin[a], b1 = a + 1 < m ? begin[a + 1] : N;
        count[a] = (int32_t)(b1 - b0);
        const uint32_t qmax = (uint32_t)(X.W - 1);
        uint32_t lo[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, hi[3] = {0, 0, 0};
        for (int64_t k = b0; k < b1; k += 4) {       // four particles' loads in flight (the last one repeats)
            double w[4][3];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) w[u][ax] = pos_s[ax * N + (k + u < b1 ? k + u : b1 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) {
                    const uint32_t q = quantise_w(w[u][ax], X.L, X.qscale, qmax);
                    lo[ax] = q < lo[ax] ? q : lo[ax];
                    hi[ax] = q > hi[ax] ? q : hi[ax];
                }
        }
        for (int ax = 0; ax < 3; ++ax) {
            B.lo[ax] = (int32_t)lo[ax];
            B.hi[ax] = (int32_t)hi[ax] + 1;
        }
        nodes[T.off[0] + i] = B;
    }
    s_box[t] = B;
    __syncthreads();
    int n = kTreeGroup;
    for (int h = 1; h <= 3; ++h) {
        n /= 8;
        IBox P;
        if (t < n) {
            P = s_box[8 * t];
            for (int c = 1; c < 8; ++c) {
                const IBox C = s_box[8 * t + c];     // empty past the last node
                for (int ax = 0; ax < 3; ++ax) {
                    P.lo[ax] = C.lo[ax] < P.lo[ax] ? C.lo[ax] : P.lo[ax];
                    P.hi[ax] = C.hi[ax] > P.hi[ax] ? C.hi[ax] : P.hi[ax];
                }
            }
            const int64_t node = (g - gp[x]) * n + t;
            if (node < T.cnt[h]) nodes[T.off[h] + node] = P;
        }
        __syncthreads();
        if (t < n) s_box[t] = P;
        __syncthreads();
    }
}

// Levels 4 and up, one workgroup per box.
__global__ void __launch_bounds__(256) tree_top_kernel(const TreeView* __restrict__ tvs,
                                                       IBox* __restrict__ nodes) {
    const TreeView& T = tvs[blockIdx.x];
    for (int h = 4; h < T.nlev; ++h) {
        const int64_t n = T.cnt[h], nchild = T.cnt[h - 1];
        const IBox* child = nodes + T.off[h - 1];
        for (int64_t i = threadIdx.x; i < n; i += blockDim.x) {
            IBox P = child[8 * i];
            const int64_t e = 8 * i + 8 < nchild ? 8 * i + 8 : nchild;
            for (int64_t c = 8 * i + 1; c < e; ++c) {
                const IBox C = child[c];
                for (int ax = 0; ax < 3; ++ax) {
                    P.lo[ax] = C.lo[ax] < P.lo[ax] ? C.lo[ax] : P.lo[ax];
                    P.hi[ax] = C.hi[ax] > P.hi[ax] ? C.hi[ax] : P.hi[ax];
                }
            }
            nodes[T.off[h] + i] = P;
        }
        __threadfence_block();
        __syncthreads();
    }
}

// Tree shapes of several boxes from their leaf counts (one workgroup).  Level
// h of all boxes is contiguous, boxes in order: lp[h (nbox + 1) + x] is the
// number of level-h nodes of the boxes before x, and the levels follow one
// another; gp[x]: the kTreeGroup-leaf groups of the boxes before x.
__global__ void __launch_bounds__(256) tree_views_kernel(const int64_t* __restrict__ loff, int nbox,
                                                         TreeView* __restrict__ tv,
                                                         int64_t* __restrict__ lp,
                                                         int64_t* __restrict__ gp, int64_t start_nodes,
                                                         int64_t* __restrict__ sizes) {
    __shared__ int64_t wsum[4];
    __shared__ int s_start;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int per = (nbox + 255) / 256;
    const int x0 = t * per < nbox ? t * per : nbox;
    const int x1 = x0 + per < nbox ? x0 + per : nbox;
    if (t == 0) s_start = 0;
    __syncthreads();
    // exclusive scan of the 256 thread sums: inside each wave, then the four
    // wave totals
    auto scan = [&](int64_t sum, int64_t* all) {
        int64_t inc = sum;
        for (int d = 1; d < 64; d <<= 1) {
            const int64_t u = __shfl_up(inc, d);
            if (lane >= d) inc += u;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        int64_t before = 0;
        *all = 0;
        for (int k = 0; k < 4; ++k) {
            if (k < wave) before += wsum[k];
            *all += wsum[k];
        }
        __syncthreads();                  // wsum is rewritten by the next scan
        return before + inc - sum;
    };
    {
        int64_t sum = 0, all = 0;
        for (int x = x0; x < x1; ++x) sum += (loff[x + 1] - loff[x] + kTreeGroup - 1) / kTreeGroup;
        int64_t acc = scan(sum, &all);
        for (int x = x0; x < x1; ++x) {
            gp[x] = acc;
            acc += (loff[x + 1] - loff[x] + kTreeGroup - 1) / kTreeGroup;
        }
        if (t == 0) gp[nbox] = all;
    }
    int64_t base = 0;                     // first node of level h (same in every thread)
    int h = 0;
    for (; h < kTreeMaxLevels; ++h) {
        int64_t sum = 0;
        for (int x = x0; x < x1; ++x) sum += level_count(loff[x + 1] - loff[x], h);
        int64_t level_total = 0;
        int64_t acc = scan(sum, &level_total);     // nodes of this level before box x0
        for (int x = x0; x < x1; ++x) {
            const int64_t c0 = loff[x + 1] - loff[x];
            const int64_t c = level_count(c0, h);
            lp[(int64_t)h * (nbox + 1) + x] = acc;
            TreeView& T = tv[x];
            if (h == 0) {
                int nl = 0;
                while (nl < kTreeMaxLevels && level_count(c0, nl) > 0) ++nl;
                T.nlev = c0 > 0 ? nl : 0;
                T.loff = loff[x];
                T.start = start_level(c0, start_nodes);
                atomicMax(&s_start, T.start);
            }
            T.cnt[h] = c;
            T.off[h] = c > 0 ? base + acc : 0;
            acc += c;
        }
        if (t == 0) lp[(int64_t)h * (nbox + 1) + nbox] = level_total;
        base += level_total;
        if (level_total == 0) break;      // no box has nodes here or above
    }
    // the levels above the last populated one: empty
    for (++h; h < kTreeMaxLevels; ++h) {
        for (int x = x0; x < x1; ++x) {
            lp[(int64_t)h * (nbox + 1) + x] = 0;
            tv[x].cnt[h] = 0;
            tv[x].off[h] = 0;
        }
        if (t == 0) lp[(int64_t)h * (nbox + 1) + nbox] = 0;
    }
    __syncthreads();
    if (t == 0) sizes[kStart] = s_start;
}

// Mass and mass-weighted position sums of every tree node (x, y, z: sum of
// m x; w: sum of m), FP64, for monopole acceptance.  Level 0 from the
// particles of each leaf, in order; level h from its (up to 8) children.
__global__ void leaf_moment_kernel(const double* __restrict__ pos_s, const float* __restrict__ mass_s,
                                   int64_t N, const int64_t* __restrict__ begin,
                                   const int64_t* __restrict__ sizes, double4* __restrict__ mc) {
    const int64_t m = sizes[kNLeaf];
    for (int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; a < m;
         a += (int64_t)gridDim.x * blockDim.x) {
    const int64_t b0 = begin[a], b1 = a + 1 < m ? begin[a + 1] : N;
    double sx = 0, sy = 0, sz = 0, sm = 0;
    for (int64_t k = b0; k < b1; ++k) {
        const double mk = (double)mass_s[k];
        sx += mk * pos_s[k];
        sy += mk * pos_s[N + k];
        sz += mk * pos_s[2 * N + k];
        sm += mk;
    }
    mc[a] = make_double4(sx, sy, sz, sm);
    }
}

__global__ void tree_moment_kernel(const TreeView* __restrict__ tv, const int64_t* __restrict__ lp,
                                   int nbox, int h, double4* __restrict__ mc) {
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < lp[nbox];
         g += (int64_t)gridDim.x * blockDim.x) {
    const int x = box_of(lp, nbox, g);
    const TreeView& T = tv[x];
    const int64_t i = g - lp[x];
    const int64_t nchild = T.cnt[h - 1];
    const double4* child = mc + T.off[h - 1];
    double4 P = child[8 * i];
    const int64_t e = 8 * i + 8 < nchild ? 8 * i + 8 : nchild;
    for (int64_t c = 8 * i + 1; c < e; ++c) {
        const double4 C = child[c];
        P.x += C.x;
        P.y += C.y;
        P.z += C.z;
        P.w += C.w;
    }
    mc[T.off[h] + i] = P;
    }
}

// ------------------------------------------------------------ box tests --
// Gap along one axis between target [loA, hiA) and source [loB, hiB)
// shifted by s * W (grid units).  Coordinates and W are at most 2^21, so
// gaps fit 32 bits and their squares one 32 x 32 -> 64 bit multiply-add.
__device__ __forceinline__ int32_t axis_gap(int32_t loA, int32_t hiA, int32_t loB, int32_t hiB, int32_t sh) {
    const int32_t g1 = loB + sh - hiA, g2 = loA - hiB - sh;
    const int32_t g = g1 > g2 ? g1 : g2;
    return g > 0 ? g : 0;
}

__device__ __forceinline__ int64_t square_add(int32_t g, int64_t r) { return (int64_t)g * g + r; }

__device__ __forceinline__ int64_t gap2_shift(const IBox& A, const IBox& B, const int s[3],
                                              int64_t W) {
    int64_t r = 0;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax)
        r = square_add(axis_gap(A.lo[ax], A.hi[ax], B.lo[ax], B.hi[ax], s[ax] * (int32_t)W), r);
    return r;
}

// Largest squared separation of the two boxes (every pair of points is
// closer): when it is below T every leaf under B passes the gap test.
__device__ __forceinline__ int64_t maxd2_shift(const IBox& A, const IBox& B, const int s[3],
                                               int64_t W) {
    int64_t r = 0;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int32_t sh = s[ax] * (int32_t)W;
        const int32_t d1 = B.hi[ax] + sh - A.lo[ax];
        const int32_t d2 = A.hi[ax] - B.lo[ax] - sh;
        r = square_add(d1 > d2 ? d1 : d2, r);
    }
    return r;
}

// Allowed shifts per axis: bit 0 -> -1, bit 1 -> 0, bit 2 -> +1.
__device__ __forceinline__ void allowed_shifts(const IBox& A, int64_t W, int64_t T, int mask[3]) {
    for (int ax = 0; ax < 3; ++ax) {
        const int64_t lo = A.lo[ax], up = W - A.hi[ax];
        mask[ax] = 2 | (lo * lo < T ? 1 : 0) | (up * up < T ? 4 : 0);
    }
}

__device__ __forceinline__ bool shift_allowed(const int mask[3], const int s[3]) {
    return (mask[0] >> (s[0] + 1) & 1) && (mask[1] >> (s[1] + 1) & 1) && (mask[2] >> (s[2] + 1) & 1);
}

__device__ __forceinline__ void decode_shift(int sc, int s[3]) {
    s[0] = sc / 9 - 1;
    s[1] = (sc / 3) % 3 - 1;
    s[2] = sc % 3 - 1;
}

// Minimum over the allowed shifts of the squared gap (a lower bound for
// every shift), used to prune subtrees when all shifts are walked at once.
__device__ __forceinline__ int64_t gap2_min(const IBox& A, const IBox& B, const int mask[3],
                                            int64_t W) {
    int64_t r = 0;
    for (int ax = 0; ax < 3; ++ax) {
        int64_t best = INT64_MAX;
        for (int s = -1; s <= 1; ++s) {
            if (!(mask[ax] >> (s + 1) & 1)) continue;
            const int64_t g = axis_gap(A.lo[ax], A.hi[ax], B.lo[ax], B.hi[ax], s * (int32_t)W);
            best = g < best ? g : best;
        }
        r += best * best;
    }
    return r;
}

// Monopole acceptance of the node of box B (global index g) for target box
// A (block b) under shift s (sec. 3.3), every enabled test required:
//  * geometric: (A + B) / R <= theta with A, B the longest box sides and R
//    the distance of the box centres, tested as (2 (A + B))^2 <= theta^2
//    (2R)^2 from integer half-cell coordinates (for theta < 1 this gives
//    B / (R - A) <= theta too);
//  * relative (Gadget-2, sec. 3.1): G M B^2 / r^4 <= alpha |a| with M the
//    node mass, r the gap between the boxes and |a| the smallest reference
//    acceleration of the block's targets, squared on both sides so that no
//    root is taken.
// Each side is a fixed sequence of FP64 operations on exact integers, the
// node mass and the block's |a|^2, so the oracle can repeat the decision.
struct MonoDev {
    double theta2, alpha;
    const double4* mc;
    const double* amin2;
};

__device__ __forceinline__ bool accept_monopole(const IBox& A, const IBox& B, const int s[3], int64_t W,
                                                const MonoDev& M, int64_t g, int64_t b, double G,
                                                double cell) {
#pragma clang fp contract(off)
    int64_t a = 0, bm = 0, r2 = 0;
    for (int ax = 0; ax < 3; ++ax) {
        const int64_t sa = (int64_t)A.hi[ax] - A.lo[ax], sb = (int64_t)B.hi[ax] - B.lo[ax];
        a = sa > a ? sa : a;
        bm = sb > bm ? sb : bm;
        const int64_t d = ((int64_t)B.lo[ax] + B.hi[ax] + 2 * (int64_t)s[ax] * W) - ((int64_t)A.lo[ax] + A.hi[ax]);
        r2 += d * d;
    }
    if (M.theta2 > 0.0) {
        const double lhs = (double)(2 * (a + bm));
        if (!(lhs * lhs <= M.theta2 * (double)r2)) return false;
    }
    if (M.alpha > 0.0) {
        const int64_t gap2 = gap2_shift(A, B, s, W);
        const double bc = (double)bm * cell;
        const double lhs = ((G * M.mc[g].w) * bc) * bc;
        const double g2 = ((double)gap2 * cell) * cell;
        const double rhs2 = ((M.alpha * M.alpha) * M.amin2[b]) * ((g2 * g2) * (g2 * g2));
        if (!(lhs * lhs <= rhs2)) return false;
    }
    return true;
}

// Smallest |a_ref|^2 over each block's targets (a_ref in input order), one
// wave per block; a value that is not a number counts only as the first.  (A
// thread per block: 244 us on 4 M particles; so: 204, bound by the gather.)
__global__ void __launch_bounds__(256) block_amin_kernel(const int32_t* __restrict__ bstart,
                                                         const int32_t* __restrict__ bcount,
                                                         const int32_t* __restrict__ perm,
                                                         const float* __restrict__ acc_ref, int64_t N,
                                                         const int64_t* __restrict__ sizes,
                                                         double* __restrict__ amin2) {
#pragma clang fp contract(off)
    const int64_t b = (int64_t)blockIdx.x * (blockDim.x / kBlock) + threadIdx.x / kBlock;
    const int lane = threadIdx.x % kBlock;
    if (b >= sizes[kNBlock]) return;
    const int32_t n = bcount[b];
    const int64_t i = perm[(int64_t)bstart[b] + (lane < n ? lane : 0)];
    const double x = (double)acc_ref[i], y = (double)acc_ref[N + i], z = (double)acc_ref[2 * N + i];
    double v = ((x * x) + (y * y)) + (z * z);
    const bool nan0 = lane == 0 && v != v;
#pragma unroll
    for (int d = 1; d < kBlock; d <<= 1) v = fmin(v, __shfl_xor(v, d));
    if (lane == 0) amin2[b] = nan0 ? (double)NAN : v;
}

// ------------------------------------------------------- canonical list --
// Depth-first walk of one tree in ascending leaf order.  test(B) decides
// whether to descend into / visit node box B; visit(leaf) is called for
// every leaf that passes.
template <class Test, class Visit>
__device__ void walk(const TreeView& tv, const IBox* nodes, Test&& test, Visit&& visit) {
    int h = tv.nlev - 1;
    int64_t i = 0;
    for (;;) {
        const bool pass = test(nodes[tv.off[h] + i]);
        if (pass && h == 0) visit(i);
        if (pass && h > 0) {
            h -= 1;
            i *= 8;
            continue;
        }
        for (;;) {
            if (h == tv.nlev - 1) return;
            const int64_t nx = i + 1;
            if ((nx & 7) != 0 && nx < tv.cnt[h]) {
                i = nx;
                break;
            }
            i >>= 3;
            h += 1;
        }
    }
}

// One thread per target leaf, all shifts in one walk, entries emitted in
// ascending (source, code) order.
template <bool FILL>
__global__ void canon_kernel(TreeView tv, const IBox* __restrict__ nodes, int64_t nleaf, int64_t W,
                             int64_t T, int32_t* __restrict__ cnt, const int64_t* __restrict__ off,
                             int32_t* __restrict__ src, uint8_t* __restrict__ code) {
    const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= nleaf) return;
    const IBox A = nodes[tv.off[0] + a];
    int mask[3];
    allowed_shifts(A, W, T, mask);
    int64_t k = FILL ? off[a] : 0;
    int32_t c = 0;
    walk(
        tv, nodes, [&](const IBox& B) { return gap2_min(A, B, mask, W) < T; },
        [&](int64_t b) {
            const IBox B = nodes[tv.off[0] + b];
            for (int sc = 0; sc < 27; ++sc) {
                int s[3];
                decode_shift(sc, s);
                if (!shift_allowed(mask, s)) continue;
                if (gap2_shift(A, B, s, W) < T) {
                    if (FILL) {
                        src[k] = (int32_t)b;
                        code[k] = (uint8_t)sc;
                        ++k;
                    } else {
                        ++c;
                    }
                }
            }
        });
    if (!FILL) cnt[a] = c;
}

// -------------------------------------------------------- target blocks --
// Minimum over the wave, in every lane: DPP steps inside the rows of 16, then
// across the rows (lane 63 holds the whole).
__device__ __forceinline__ int32_t wave_min_i(int32_t v) {
#define PP_DPP_MIN(ctrl, rows)                                                             \
    {                                                                                      \
        const int32_t o = __builtin_amdgcn_update_dpp(INT32_MAX, v, ctrl, rows, 0xf, false); \
        v = o < v ? o : v;                                                                 \
    }
    PP_DPP_MIN(0x111, 0xf)               // row_shr:1
    PP_DPP_MIN(0x112, 0xf)               // row_shr:2
    PP_DPP_MIN(0x114, 0xf)               // row_shr:4
    PP_DPP_MIN(0x118, 0xf)               // row_shr:8
    PP_DPP_MIN(0x142, 0xa)               // row_bcast:15
    PP_DPP_MIN(0x143, 0xc)               // row_bcast:31
#undef PP_DPP_MIN
    return __builtin_amdgcn_readlane(v, 63);
}

// One wave per chunk of kBlock consecutive particles of one box.  Every lane
// quantises its particle; if the chunk's bounding box is at most emax grid
// units wide along every axis (the common case) the chunk is one block.
// Otherwise lane 0 walks the chunk and starts a new block whenever adding the
// next particle would make the box wider than emax.
struct Chunk {
    int64_t k0, k1;                      // its particles
    int x;                               // its box
};
__device__ __forceinline__ Chunk chunk_of(const BatchDev& bd, const int64_t* __restrict__ choff, int64_t c) {
    Chunk r;
    r.x = box_of(choff, bd.nbox, c);
    const BoxDev& X = bd.box[r.x];
    r.k0 = X.poff + (c - choff[r.x]) * kBlock;
    const int64_t kend = X.poff + X.n;
    r.k1 = r.k0 + kBlock < kend ? r.k0 + kBlock : kend;
    return r;
}

// The chunk's bounding box; whether it is one block.
__device__ __forceinline__ bool chunk_fits(const BoxDev& X, const double* __restrict__ pos_s, int64_t N,
                                           const Chunk& ch, IBox& B) {
    const uint32_t qmax = (uint32_t)(X.W - 1);
    const int64_t k = ch.k0 + (threadIdx.x & (kBlock - 1));
    const bool valid = k < ch.k1;
    double w[3];
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) w[ax] = valid ? pos_s[ax * N + k] : 0.0;
    bool fits = true;
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int32_t q = (int32_t)quantise_w(w[ax], X.L, X.qscale, qmax);
        B.lo[ax] = wave_min_i(valid ? q : INT32_MAX);
        B.hi[ax] = -wave_min_i(valid ? -q - 1 : INT32_MAX);
        fits = fits && (int64_t)(B.hi[ax] - B.lo[ax]) <= X.emax;
    }
    return fits;
}

// The walk of a wide chunk: the number of its blocks (lane 0), each handed to
// write(number, first particle, end, box).  qs: this wave's LDS.
template <class Write>
__device__ __forceinline__ int32_t chunk_walk(const BoxDev& X, const double* __restrict__ pos_s, int64_t N,
                                              const Chunk& ch, int32_t (*qs)[kBlock], Write&& write) {
    const int lane = threadIdx.x & (kBlock - 1);
    const uint32_t qmax = (uint32_t)(X.W - 1);
    const bool valid = ch.k0 + lane < ch.k1;
    wave_sync();                         // lane 0 is done with the previous chunk
    for (int ax = 0; ax < 3; ++ax)
        qs[ax][lane] = valid ? (int32_t)quantise_w(pos_s[ax * N + ch.k0 + lane], X.L, X.qscale, qmax) : 0;
    wave_sync();
    int32_t nb = 0;
    if (lane != 0) return 0;
    int64_t start = ch.k0;
    IBox B;
    for (int64_t kk = ch.k0; kk < ch.k1; ++kk) {
        const int l = (int)(kk - ch.k0);
        const int32_t q[3] = {qs[0][l], qs[1][l], qs[2][l]};
        IBox U = B;
        bool wide = kk == ch.k0;
        if (!wide)
            for (int ax = 0; ax < 3; ++ax) {
                U.lo[ax] = q[ax] < U.lo[ax] ? q[ax] : U.lo[ax];
                U.hi[ax] = q[ax] + 1 > U.hi[ax] ? q[ax] + 1 : U.hi[ax];
                wide |= (int64_t)(U.hi[ax] - U.lo[ax]) > X.emax;
            }
        if (wide) {
            if (kk > ch.k0) write(nb++, start, kk, B);
            start = kk;
            for (int ax = 0; ax < 3; ++ax) {
                B.lo[ax] = q[ax];
                B.hi[ax] = q[ax] + 1;
            }
        } else {
            B = U;
        }
    }
    write(nb++, start, ch.k1, B);
    return nb;
}

struct BlockOut {
    int32_t* bstart;
    int32_t* bcount;
    IBox* box;
    int32_t* bboxid;
    int64_t cap;
    __device__ __forceinline__ void put(int64_t at, int64_t from, int64_t to, const IBox& B, int x) const {
        if (at >= cap) return;           // too many blocks: reported by the count
        bstart[at] = (int32_t)from;
        bcount[at] = (int32_t)(to - from);
        box[at] = B;
        bboxid[at] = x;
    }
};

// Many chunks: a counting launch that leaves every chunk's box (in the
// `cbox`) beside its number of blocks, a scan, and a writing launch that
// reads positions again for the wide chunks only.  (2.1 M particles: 59 us of
// kernels, 62 when both launches read all positions, 74 in the one-launch form
// below, whose workgroups wait for one another.)
template <bool FILL>
__global__ void __launch_bounds__(256) block_split_kernel(BatchDev bd, const double* __restrict__ pos_s, int64_t N,
                                                          const int64_t* __restrict__ choff, int64_t nchunk,
                                                          int32_t* __restrict__ ccount,
                                                          const int64_t* __restrict__ coff,
                                                          IBox* __restrict__ cbox, BlockOut out) {
    __shared__ int32_t qs[256 / kBlock][3][kBlock];
    const int wave = threadIdx.x / kBlock;
    const bool first = (threadIdx.x & (kBlock - 1)) == 0;
    const int64_t c = (int64_t)blockIdx.x * (256 / kBlock) + wave;
    if (c >= nchunk) return;
    const Chunk ch = chunk_of(bd, choff, c);
    const BoxDev& X = bd.box[ch.x];
    if (!FILL) {
        IBox B;
        int32_t nb = 1;
        if (!chunk_fits(X, pos_s, N, ch, B))
            nb = chunk_walk(X, pos_s, N, ch, qs[wave], [](int32_t, int64_t, int64_t, const IBox&) {});
        if (!first) return;
        ccount[c] = nb;
        cbox[c] = B;
        return;
    }
    const int64_t o = coff[c];
    if (ccount[c] == 1) {
        if (first) out.put(o, ch.k0, ch.k1, cbox[c], ch.x);
        return;
    }
    chunk_walk(X, pos_s, N, ch, qs[wave], [&](int32_t i, int64_t from, int64_t to, const IBox& B) {
        out.put(o + i, from, to, B, ch.x);
    });
}

// Few chunks (kFewChunks): one launch counts, scans (running sums of the workgroup and
// look-back over the earlier ones) and writes.
constexpr int kSplitWaves = 8;

__global__ void __launch_bounds__(64 * kSplitWaves) block_split_small_kernel(
    BatchDev bd, const double* __restrict__ pos_s, int64_t N, const int64_t* __restrict__ choff,
    int64_t nchunk, LbArgs lb, int64_t ntile, int64_t* __restrict__ coff, int64_t* __restrict__ sizes,
    BlockOut out) {
    __shared__ int32_t qs[kSplitWaves][3][kBlock];
    __shared__ int32_t s_cnt[kSplitWaves];
    __shared__ unsigned s_tile;
    __shared__ int64_t s_pre;
    const int lane = threadIdx.x & (kBlock - 1), wave = threadIdx.x / kBlock;
    lb_clear_other(lb);
    if (threadIdx.x == 0) s_tile = (unsigned)atomicAdd(lb.cur, 1ull);
    __syncthreads();
    const int64_t tile = s_tile, c = tile * kSplitWaves + wave;
    const bool any = c < nchunk;
    Chunk ch{};
    IBox B;
    bool fits = false;
    int32_t nb = 0;
    if (any) {
        ch = chunk_of(bd, choff, c);
        fits = chunk_fits(bd.box[ch.x], pos_s, N, ch, B);
        nb = fits ? 1
                  : chunk_walk(bd.box[ch.x], pos_s, N, ch, qs[wave], [](int32_t, int64_t, int64_t, const IBox&) {});
    }
    if (lane == 0) s_cnt[wave] = nb;
    __syncthreads();
    if (wave == 0) {
        int64_t agg = 0;
        for (int k = 0; k < kSplitWaves; ++k) agg += s_cnt[k];
        const int64_t ex = lb_tile_prefix<1>(lb, tile, 0, agg, sizes, lane);
        if (lane == 0) {
            s_pre = ex;
            if (tile == ntile - 1) {
                const int64_t total = ex + agg;
                coff[nchunk] = total;
                sizes[kNeedBlock] = total;
                sizes[kNBlock] = total < out.cap ? total : out.cap;
                if (total > out.cap) atomicOr(reinterpret_cast<unsigned long long*>(sizes + kOverflow), 1ull);
            }
        }
    }
    __syncthreads();
    if (!any) return;
    int64_t o = s_pre;
    for (int k = 0; k < wave; ++k) o += s_cnt[k];
    if (lane == 0) coff[c] = o;
    if (fits) {
        if (lane == 0) out.put(o, ch.k0, ch.k1, B, ch.x);
        return;
    }
    chunk_walk(bd.box[ch.x], pos_s, N, ch, qs[wave], [&](int32_t i, int64_t from, int64_t to, const IBox& U) {
        out.put(o + i, from, to, U, ch.x);
    });
}

// ----------------------------------------------------------- block lists --
// A node passes for target box A under shift s when its box is closer than
// r_cut (gap^2 < T); it is *inside* when even its farthest point is
// (maxdist^2 < T), and then every leaf under it passes, so the node's whole
// leaf interval is listed without descending.  One wave per block
// first tests the nodes of the box's start level (TreeView::start, few nodes)
// and those above them; the walk is then level-synchronous down to level 2
// over all (block, shift, node) entries
// at once (one thread per entry, children written in order so entries stay
// sorted by block, shift, node); then one thread per entry walks its
// subtree (at most 64 leaves) depth-first, testing the 8 children of a node
// at once.  While the entries stay within a memory budget the breadth-first
// part goes one level further (down to level 1), which leaves a single
// 8-child test per entry.  Leaves (or inside intervals) come in ascending order and
// consecutive ones merge into one range of source particles.
constexpr int kDfsLevel = 2;
// A box that lists fewer than kSmallBox sources in all is cut into chunks of
// kChunkScale listed^(2/3) positions: an item's fixed cost grows with the
// number of items (listed / chunk), the wait for the last items with the
// chunk.  Measured fastest chunks (PP stage, one wave per block): 1000
// particles (49 k listed) 64, 28 us against 189 at 2048; 20 k (1.3 M) 128, 65
// against 142; 32 k (2 M) 128, 85 against 155; 150 k (10 M) 256, 246 against
// 350; 300 k (20 M) 256 to 512, 454 against 535; 1 M (70 M) 1024, 1.44 ms
// against 1.50.  The rule stays at or above them; its floors cost a lone box 1
// to 5 us.  A batch waits for its last items once, however many boxes it has, so
// all of it together is cut into no more than kEnoughItems by this rule: with
// each box cut as if it were alone 20000 boxes of 1000 particles took 35.2 ms
// against 30.6 at 2048 positions, 4000 of them 7.36 against 6.48, 1000 boxes of
// 32 k 66.6 against 62.0, 64 of 100 k 15.3 against 14.8.  A lone box is never
// bounded by it (2^27 positions in 65536 items are 2048 each).
constexpr int64_t kSmallBox = (int64_t)1 << 27;
constexpr double kChunkScale = 0.01075;
constexpr int64_t kTinyBox = (int64_t)1 << 17;
constexpr int64_t kTinyChunk = 128, kSmallChunk = 256;
constexpr int64_t kEnoughItems = 65536;
// target blocks per box up to which the first guess of the items follows that rule
constexpr int64_t kSmallBlocks = 65536;
// Monopoles may be taken at every level: by the breadth-first expansion for
// nodes of level 2 and up, by the depth-first walk for groups of 8 leaves
// (level 1) and single leaves (level 0).
constexpr int kMonoMinLevel = 0;


// Test the children of (h, i): pass bits and inside bits (inside implies pass).
__device__ __forceinline__ void expand2(const TreeView& tv, const IBox* nodes, int h, int64_t i,
                                        const IBox& A, const int s[3], int64_t W, int64_t T,
                                        uint32_t& pass, uint32_t& inside) {
    const int64_t c0 = 8 * i, nc = tv.cnt[h - 1];
    const int n = nc - c0 < 8 ? (int)(nc - c0) : 8;
    // all 8 boxes at once (past the last child: nodes of the next level, or the 8
    // boxes that tree_node_bound adds), so that their loads overlap: child by
    // child, 164 us in the range count on 2.1 M particles, so 136
    IBox C[8];
    __builtin_memcpy(C, nodes + tv.off[h - 1] + c0, sizeof(C));
    pass = 0;
    inside = 0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const bool in = c < n && gap2_shift(A, C[c], s, W) < T;
        pass |= in ? 1u << c : 0u;
        inside |= in && maxd2_shift(A, C[c], s, W) < T ? 1u << c : 0u;
    }
}

// The first entries of a block: for every allowed shift, the nodes of the
// box's start level that pass, 64 at a time and in order.  A node that passes
// has ancestors that pass, so those need no test of their own but for
// monopoles: then they are tested from the root down, and an accepted one
// becomes the entry itself, written by its first node of the start level.  The
// entries are those of a walk from the root, which took two kernels and a scan
// per level.
//
// One wave walks the units (allowed shift, 64 nodes) from u0 to u1 - 1 of
// block b and returns the number of entries, which it writes from number o on
// when `fill`.  With KEEP, the first KEEP units' ballots of the counting walk
// stay in `keep` (LDS) for the writing one, which then visits the passing nodes
// only.
template <int KEEP>
__device__ __forceinline__ int32_t start_walk(const TreeView& tv, const BoxDev& X, const IBox* __restrict__ nodes,
                                              const IBox& A, int64_t b, const int mask[3], int u0, int u1,
                                              bool fill, int64_t o, FEntry* __restrict__ out, int64_t cap_out,
                                              const MonoDev& mono, uint64_t* keep) {
    const int lane = threadIdx.x & (kBlock - 1);
    const int64_t W = X.W, T = X.T;
    const int top = tv.nlev - 1, start = tv.start;
    const int64_t n0 = tv.cnt[start];
    const int per = (int)((n0 + kBlock - 1) / kBlock);               // units per shift
    const bool mono_on = mono.theta2 > 0.0 || mono.alpha > 0.0;
    // with monopoles the first unit of every higher node is walked in any case:
    // such a node may lie within the cut, and be accepted, where its first 64
    // nodes do not, and the entry is theirs to write
    const bool higher = mono_on && start + 3 <= top;
    int32_t c = 0;
    int u = 0;
    for (int sc = 0; sc < 27 && u < u1; ++sc) {
        int s[3];
        decode_shift(sc, s);
        if (!shift_allowed(mask, s)) continue;
        if (u + per <= u0) {
            u += per;
            continue;
        }
        for (int i = 0; i < per; ++i, ++u) {
            if (u < u0 || u >= u1) continue;
            const bool kept = u - u0 < KEEP;
            uint64_t known = ~0ull;
            if (fill && kept) {
                known = keep[u - u0];
                if (known == 0) continue;
            }
            const int64_t node = (int64_t)i * kBlock + lane;
            FEntry E{};
            bool emit = false;
            // the 64 nodes' common ancestor first (its box holds theirs)
            if ((fill && kept) || start + 2 > top || gap2_shift(A, nodes[tv.off[start + 2] + i], s, W) < T ||
                (higher && (i & 7) == 0))
                for (int h = mono_on ? top : start; h >= start && node < n0 && (known >> lane & 1ull); --h) {
                    const int64_t up = node >> (3 * (h - start));
                    const IBox R = nodes[tv.off[h] + up];
                    if (!(gap2_shift(A, R, s, W) < T)) break;
                    const bool taken = mono_on && h >= kMonoMinLevel &&
                                       accept_monopole(A, R, s, W, mono, tv.off[h] + up, b, X.G, X.cell);
                    if (h > start && !taken) continue;
                    E.blk = (int32_t)b;
                    E.node = (int32_t)up;
                    E.sc = (uint8_t)sc;
                    E.lev = (uint8_t)h;
                    E.inside = fill && maxd2_shift(A, R, s, W) < T;
                    E.mono = taken;
                    emit = up << (3 * (h - start)) == node;
                    break;
                }
            const uint64_t bal = __ballot(emit);
            if (KEEP > 0 && !fill && kept && lane == 0) keep[u - u0] = bal;
            if (fill) {
                const int64_t at = o + c + __popcll(bal & ((1ull << lane) - 1ull));
                if (emit && at < cap_out) out[at] = E;
            }
            c += __popcll(bal);
        }
    }
    return c;
}

// A box that every lane holds alike, in scalar registers.
__device__ __forceinline__ IBox uniform_box(const IBox& B) {
    IBox r;
    for (int ax = 0; ax < 3; ++ax) {
        r.lo[ax] = __builtin_amdgcn_readfirstlane(B.lo[ax]);
        r.hi[ax] = __builtin_amdgcn_readfirstlane(B.hi[ax]);
    }
    return r;
}

__device__ __forceinline__ int start_units(const TreeView& tv, const int mask[3]) {
    return __popc(mask[0]) * __popc(mask[1]) * __popc(mask[2]) * (int)((tv.cnt[tv.start] + kBlock - 1) / kBlock);
}

// Large boxes, up to kManyBlocks blocks: one wave per block, a counting and a
// writing launch around a scan.
template <bool FILL>
__global__ void __launch_bounds__(256) start_kernel(BatchDev bd, const TreeView* __restrict__ tvs,
                                                    const IBox* __restrict__ nodes,
                                                    const IBox* __restrict__ bbox,
                                                    const int32_t* __restrict__ bboxid,
                                                    const int64_t* __restrict__ sizes, int64_t cap_in,
                                                    int32_t* __restrict__ cnt, const int64_t* __restrict__ off,
                                                    FEntry* __restrict__ out, int64_t cap_out, MonoDev mono) {
    const int64_t b = (int64_t)blockIdx.x * (256 / kBlock) + __builtin_amdgcn_readfirstlane((int)threadIdx.x / kBlock);
    if (b >= cap_in) return;
    const bool first = (threadIdx.x & (kBlock - 1)) == 0;
    if (b >= sizes[kNBlock]) {
        if (!FILL && first) cnt[b] = 0;
        return;
    }
    const int x = __builtin_amdgcn_readfirstlane(bboxid[b]);
    const IBox A = uniform_box(bbox[b]);
    int mask[3];
    allowed_shifts(A, bd.box[x].W, bd.box[x].T, mask);
    const int32_t c = start_walk<0>(tvs[x], bd.box[x], nodes, A, b, mask, 0, start_units(tvs[x], mask), FILL,
                                    FILL ? off[b] : 0, out, cap_out, mono, nullptr);
    if (!FILL && first) cnt[b] = c;
}

// The same with one lane per block, for more than kManyBlocks of them: each
// lane walks its box's tree from the root down to the start level, in order.
// Neighbouring blocks take nearly the same way.  A wave per block tests every
// node of the start level, most lanes of it idle, and costs about 1 us of a
// wave's time for each block: 4 M particles whose cut splits them into 1.6 M
// blocks took 1122 us in both launches, so 182; 16.8 M clustered ones 575, so
// 152; 64 boxes of a batch (500 k blocks) 1198, so 454; 63 k blocks with
// monopoles 269, so 199.  Fewer blocks leave lanes without enough waves in
// flight: 37 k of them 94, so 162.
template <bool FILL>
__global__ void __launch_bounds__(256) start_many_kernel(BatchDev bd, const TreeView* __restrict__ tvs,
                                                         const IBox* __restrict__ nodes,
                                                         const IBox* __restrict__ bbox,
                                                         const int32_t* __restrict__ bboxid,
                                                         const int64_t* __restrict__ sizes, int64_t cap_in,
                                                         int32_t* __restrict__ cnt, const int64_t* __restrict__ off,
                                                         FEntry* __restrict__ out, int64_t cap_out, MonoDev mono) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= cap_in) return;
    if (b >= sizes[kNBlock]) {
        if (!FILL) cnt[b] = 0;
        return;
    }
    const int x = bboxid[b];
    const TreeView& tv = tvs[x];
    const BoxDev& X = bd.box[x];
    const IBox A = bbox[b];
    const int64_t W = X.W, T = X.T;
    const int top = tv.nlev - 1, start = tv.start;
    const bool mono_on = mono.theta2 > 0.0 || mono.alpha > 0.0;
    int mask[3];
    allowed_shifts(A, W, T, mask);
    int64_t o = FILL ? off[b] : 0;
    int32_t c = 0;
    for (int sc = 0; sc < 27; ++sc) {
        int s[3];
        decode_shift(sc, s);
        if (!shift_allowed(mask, s)) continue;
        int h = top;
        int64_t i = 0;
        for (;;) {
            const int64_t g = tv.off[h] + i;
            const IBox R = nodes[g];
            if (gap2_shift(A, R, s, W) < T) {
                const bool taken = mono_on && h >= kMonoMinLevel && accept_monopole(A, R, s, W, mono, g, b, X.G, X.cell);
                if (!taken && h > start) {
                    h -= 1;
                    i *= 8;
                    continue;
                }
                if (FILL && o < cap_out) {
                    FEntry E;
                    E.blk = (int32_t)b;
                    E.node = (int32_t)i;
                    E.sc = (uint8_t)sc;
                    E.lev = (uint8_t)h;
                    E.inside = maxd2_shift(A, R, s, W) < T;
                    E.mono = taken;
                    out[o] = E;
                }
                ++o;
                ++c;
            }
            while (h < top && (((i + 1) & 7) == 0 || i + 1 >= tv.cnt[h])) {
                i >>= 3;
                h += 1;
            }
            if (h == top) break;
            ++i;
        }
    }
    if (!FILL) cnt[b] = c;
}

// Small boxes: kStartSplit waves share a block, each a stretch of its units (a
// small box has few blocks and many units: 32 k particles took 50 us with a
// wave per block, 30 so), and one launch counts, scans (look-back over the
// workgroups) and writes.  With many workgroups the look-back costs more than
// the launches it saves (2.1 M particles: 175 us against 96).
constexpr int kStartWaves = 8, kStartSplit = 4, kStartKeep = 48;

__global__ void __launch_bounds__(64 * kStartWaves) start_small_kernel(
    BatchDev bd, const TreeView* __restrict__ tvs, const IBox* __restrict__ nodes,
    const IBox* __restrict__ bbox, const int32_t* __restrict__ bboxid, LbArgs lb, int64_t ntile,
    int64_t* sizes, FEntry* __restrict__ out, int64_t cap_out, int slot2, MonoDev mono) {
    __shared__ unsigned s_tile;
    __shared__ int32_t s_cnt[kStartWaves];
    __shared__ uint64_t s_keep[kStartWaves][kStartKeep];
    __shared__ int64_t s_pre;
    const int lane = threadIdx.x & (kBlock - 1), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kBlock);
    lb_clear_other(lb);
    if (threadIdx.x == 0) s_tile = (unsigned)atomicAdd(lb.cur, 1ull);
    __syncthreads();
    const int64_t tile = __builtin_amdgcn_readfirstlane((int)s_tile);
    const int64_t b = tile * (kStartWaves / kStartSplit) + wave / kStartSplit;
    const bool any = b < sizes[kNBlock];
    const int x = any ? __builtin_amdgcn_readfirstlane(bboxid[b]) : 0;
    IBox A{};
    int mask[3] = {0, 0, 0};
    if (any) {
        A = uniform_box(bbox[b]);
        allowed_shifts(A, bd.box[x].W, bd.box[x].T, mask);
    }
    const int units = start_units(tvs[x], mask), w = wave % kStartSplit;
    const int u0 = units * w / kStartSplit, u1 = units * (w + 1) / kStartSplit;
    const int32_t mine = start_walk<kStartKeep>(tvs[x], bd.box[x], nodes, A, b, mask, u0, u1, false, 0, out,
                                                cap_out, mono, s_keep[wave]);
    if (lane == 0) s_cnt[wave] = mine;
    __syncthreads();
    if (wave == 0) {
        int64_t agg = 0;
        for (int k = 0; k < kStartWaves; ++k) agg += s_cnt[k];
        const int64_t ex = lb_tile_prefix<1>(lb, tile, 0, agg, sizes, lane);
        if (lane == 0) {
            s_pre = ex;
            if (tile == ntile - 1) {
                const int64_t total = ex + agg, kept = total < cap_out ? total : cap_out;
                sizes[kNeedEntry0] = total;
                sizes[kEntry0] = kept;
                if (slot2 >= 0) sizes[slot2] = kept;
                if (total > cap_out) atomicOr(reinterpret_cast<unsigned long long*>(sizes + kOverflow), 2ull);
            }
        }
    }
    __syncthreads();
    int64_t o = s_pre;
    for (int k = 0; k < wave; ++k) o += s_cnt[k];
    start_walk<kStartKeep>(tvs[x], bd.box[x], nodes, A, b, mask, u0, u1, true, o, out, cap_out, mono, s_keep[wave]);
}

// One level down: entries above the DFS level that are not inside are
// replaced by their passing children; the others are carried unchanged.
// The count pass keeps each opened entry's child tests (passing children in
// the low byte, inside children in the next) in cmask, and the fill pass
// reads them back instead of testing the child boxes again.
template <bool FILL>
__global__ void bfs_level_kernel(BatchDev bd, const TreeView* __restrict__ tvs,
                                 const IBox* __restrict__ nodes, const IBox* __restrict__ bbox,
                                 const int32_t* __restrict__ bboxid, const FEntry* __restrict__ in,
                                 const int64_t* __restrict__ F_in, int64_t cap_in, int stop,
                                 int32_t* __restrict__ cnt, const int64_t* __restrict__ off,
                                 FEntry* __restrict__ out, int64_t cap_out, MonoDev mono,
                                 uint16_t* __restrict__ cmask) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= cap_in) return;
    if (e >= *F_in) {
        if (!FILL) cnt[e] = 0;
        return;
    }
    const FEntry E = in[e];
    // with monopole acceptance, inside entries are opened too (a child may
    // be accepted); accepted entries are final
    const bool mono_on = mono.theta2 > 0.0 || mono.alpha > 0.0;
    if (E.mono || E.lev <= stop || (E.inside && !mono_on)) {
        if (FILL) {
            if (off[e] < cap_out) out[off[e]] = E;
        } else {
            cnt[e] = 1;
        }
        return;
    }
    const int x = bboxid[E.blk];
    int s[3];
    decode_shift(E.sc, s);
    uint32_t pass, inside;
    if (!FILL) {
        expand2(tvs[x], nodes, E.lev, E.node, bbox[E.blk], s, bd.box[x].W, bd.box[x].T, pass, inside);
        cnt[e] = __popc(pass);
        cmask[e] = (uint16_t)(pass | (inside << 8));
        return;
    }
    const uint32_t m = cmask[e];
    pass = m & 0xffu;
    inside = m >> 8;
    int64_t o = off[e];
    while (pass) {
        const int c = __builtin_ctz(pass);
        pass &= pass - 1;
        FEntry C;
        C.blk = E.blk;
        C.node = 8 * E.node + c;
        C.sc = E.sc;
        C.lev = (uint8_t)(E.lev - 1);
        C.inside = (inside >> c) & 1u;
        C.mono = mono_on && C.lev >= kMonoMinLevel &&
                 accept_monopole(bbox[E.blk], nodes[tvs[x].off[C.lev] + C.node], s, bd.box[x].W, mono,
                                 tvs[x].off[C.lev] + C.node, E.blk, bd.box[x].G, bd.box[x].cell);
        if (o < cap_out) out[o] = C;
        ++o;
    }
}

// Depth-first walk of one entry's subtree (at most 8^2 = 64 leaves).  The
// count pass records which leaves of the subtree pass as a 64-bit mask
// (bit = leaf - first leaf of the subtree); the fill pass turns the mask
// back into runs without testing boxes again, writing them from range slot
// o and list position pos.  Inside entries and leaf entries are a single
// run and need no mask.  Returns the entry's runs (nr) and sources (tot);
// with monopole acceptance on (count pass), children met by the walk are
// tested too: accepted leaves go to m0 (bit = leaf - first leaf of the
// entry), accepted groups of 8 leaves to m1 (bit = group - first group),
// and are not listed.
template <bool FILL>
__device__ void entry_ranges(const BatchDev& bd, const TreeView* __restrict__ tvs,
                             const IBox* __restrict__ nodes, const FEntry E, int64_t e,
                             const IBox* __restrict__ bbox, const int32_t* __restrict__ bboxid,
                             const int64_t* __restrict__ leaf_begin,
                             const int32_t* __restrict__ leaf_count, uint64_t* __restrict__ lmask,
                             int32_t* __restrict__ rbeg, int32_t* __restrict__ rpre,
                             uint8_t* __restrict__ rcode, const MonoDev& mono, int64_t o,
                             int64_t pos, int64_t cap_range, int32_t& nr, int64_t& tot,
                             uint64_t& m0, uint32_t& m1) {
    const int x = bboxid[E.blk];
    const TreeView& tv = tvs[x];
    const int64_t nleaf = tv.cnt[0];
    const bool mono_on = !FILL && (mono.theta2 > 0.0 || mono.alpha > 0.0);
    m0 = 0;
    m1 = 0;
    nr = 0;
    tot = 0;
    // one run of local leaves [l0, l1]
    auto emit = [&](int64_t l0, int64_t l1) {
        const int64_t p0 = leaf_begin[tv.loff + l0];
        const int64_t p1 = leaf_begin[tv.loff + l1] + leaf_count[tv.loff + l1];
        if (FILL) {
            if (o < cap_range) {
                rbeg[o] = (int32_t)p0;
                rpre[o] = (int32_t)pos;
                rcode[o] = E.sc;
            }
            ++o;
        }
        ++nr;
        pos += p1 - p0;
        tot += p1 - p0;
    };
    const int64_t first = (int64_t)E.node << (3 * E.lev);
    int64_t last = (((int64_t)E.node + 1) << (3 * E.lev)) - 1;
    if (last > nleaf - 1) last = nleaf - 1;
    const bool walk_inside = mono.theta2 > 0.0 || mono.alpha > 0.0;   // inside nodes are opened too
    if (E.mono || (E.lev > kDfsLevel && (!E.inside || walk_inside))) {
        // a monopole: no source ranges; a node above the walk's reach: the
        // pass runs again with more expansion passes (finish_items)
    } else if (E.lev == 0 || (E.inside && !walk_inside)) {
        emit(first, last);
    } else {
        uint64_t mask = 0;
        if (FILL) {
            mask = lmask[e];
        } else {
            const IBox A = bbox[E.blk];
            const int64_t W = bd.box[x].W, T = bd.box[x].T;
            int s[3];
            decode_shift(E.sc, s);
            // 16 bits per level: low byte pending children, high byte inside children
            uint64_t st = 0;
            int lev = E.lev;
            int64_t node = E.node;
            uint32_t pa, in;
            expand2(tv, nodes, lev, node, A, s, W, T, pa, in);
            st |= (uint64_t)(pa | (in << 8)) << (16 * (lev & 3));
            for (;;) {
                const uint32_t wv = (uint32_t)(st >> (16 * (lev & 3))) & 0xffffu;
                const uint32_t m = wv & 0xffu;
                if (m == 0) {
                    if (lev == E.lev) break;
                    ++lev;
                    node >>= 3;
                    continue;
                }
                const int c = __builtin_ctz(m);
                const uint32_t w2 = wv & ~(1u << c);
                st = (st & ~(0xffffull << (16 * (lev & 3)))) | ((uint64_t)w2 << (16 * (lev & 3)));
                const int64_t child = 8 * node + c;
                if (mono_on) {
                    const int64_t g = tv.off[lev - 1] + child;
                    if (accept_monopole(A, nodes[g], s, W, mono, g, E.blk, bd.box[x].G, bd.box[x].cell)) {
                        if (lev == 1) m0 |= 1ull << (child - first);
                        else m1 |= 1u << (child - (first >> 3));
                        continue;
                    }
                }
                if (lev == 1 || (!walk_inside && ((wv >> 8) >> c & 1u))) {
                    const int64_t l0 = child << (3 * (lev - 1));
                    int64_t l1 = ((child + 1) << (3 * (lev - 1))) - 1;
                    if (l1 > nleaf - 1) l1 = nleaf - 1;
                    for (int64_t l = l0; l <= l1; ++l) mask |= 1ull << (l - first);
                } else {
                    --lev;
                    node = child;
                    expand2(tv, nodes, lev, node, A, s, W, T, pa, in);
                    st = (st & ~(0xffffull << (16 * (lev & 3)))) |
                         ((uint64_t)(pa | (in << 8)) << (16 * (lev & 3)));
                }
            }
            lmask[e] = mask;
        }
        // runs of set bits, ascending
        while (mask) {
            const int a = __builtin_ctzll(mask);
            const uint64_t above = ~mask & (~0ull << a);      // first clear bit at or above a
            const int z = above ? __builtin_ctzll(above) : 64;
            emit(first + a, first + z - 1);
            mask = z >= 64 ? 0ull : mask & (~0ull << z);
        }
    }
}

// Count pass: every entry walks its subtree and records its runs (rcnt)
// and listed sources (scnt); entries past the entry count get zero.
__global__ void ranges_count_kernel(BatchDev bd, const TreeView* __restrict__ tvs,
                                    const IBox* __restrict__ nodes, const FEntry* __restrict__ ent,
                                    int64_t F, const IBox* __restrict__ bbox,
                                    const int32_t* __restrict__ bboxid,
                                    const int64_t* __restrict__ leaf_begin,
                                    const int32_t* __restrict__ leaf_count,
                                    uint64_t* __restrict__ lmask, int32_t* __restrict__ rcnt,
                                    int32_t* __restrict__ scnt, MonoDev mono,
                                    uint64_t* __restrict__ mono0, uint8_t* __restrict__ mono1,
                                    const int64_t* __restrict__ sizes) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= F) return;                       // F: the capacity of the entry buffer
    int32_t nr = 0;
    int64_t tot = 0;
    uint64_t m0 = 0;
    uint32_t m1 = 0;
    if (e < sizes[kNEntry])
        entry_ranges<false>(bd, tvs, nodes, ent[e], e, bbox, bboxid, leaf_begin, leaf_count, lmask,
                            nullptr, nullptr, nullptr, mono, 0, 0, 0, nr, tot, m0, m1);
    rcnt[e] = nr;
    scnt[e] = (int32_t)(tot < INT32_MAX ? tot : INT32_MAX);
    if (mono0) {
        mono0[e] = m0;
        mono1[e] = (uint8_t)m1;
    }
}

// First entry of every block (entries are sorted by block), and from it the
// block's first range and its list length; flags a list longer than int32.
__global__ void block_sum_kernel(const FEntry* __restrict__ ent, const int64_t* __restrict__ roff_e,
                                 const int64_t* __restrict__ soff_e, int64_t* __restrict__ sizes,
                                 int64_t cap_block, int64_t* __restrict__ eoff, int64_t* __restrict__ roff,
                                 int32_t* __restrict__ slen) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nblock = sizes[kNBlock], F = sizes[kNEntry];
    if (b > nblock || b > cap_block) return;
    int64_t lo = 0, hi = F;             // first e with ent[e].blk >= b
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (ent[mid].blk < b) lo = mid + 1;
        else hi = mid;
    }
    eoff[b] = lo;
    roff[b] = roff_e[lo];
    if (b == nblock) return;
    // the block's end: its entries are few, so the next block is found by
    // doubling from its first
    int64_t step = 64, end = lo;
    while (end + step < F && ent[end + step].blk <= b) {
        end += step;
        step *= 2;
    }
    hi = end + step < F ? end + step : F;
    lo = end;                           // first e >= lo with ent[e].blk > b
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (ent[mid].blk <= b) lo = mid + 1;
        else hi = mid;
    }
    const int64_t len = soff_e[lo] - soff_e[eoff[b]];
    if (len > INT32_MAX) atomicOr(reinterpret_cast<unsigned long long*>(sizes + kOverflow), 16ull);
    slen[b] = (int32_t)(len < INT32_MAX ? len : INT32_MAX);
}

// Fill pass: every entry writes its runs from its first range slot, with
// list positions relative to its block.
__global__ void ranges_fill_kernel(BatchDev bd, const TreeView* __restrict__ tvs,
                                   const IBox* __restrict__ nodes, const FEntry* __restrict__ ent,
                                   int64_t F, const IBox* __restrict__ bbox,
                                   const int32_t* __restrict__ bboxid,
                                   const int64_t* __restrict__ leaf_begin,
                                   const int32_t* __restrict__ leaf_count,
                                   uint64_t* __restrict__ lmask, const int64_t* __restrict__ roff_e,
                                   const int64_t* __restrict__ soff_e, const int64_t* __restrict__ eoff,
                                   int32_t* __restrict__ rbeg, int32_t* __restrict__ rpre,
                                   uint8_t* __restrict__ rcode, MonoDev mono,
                                   const int64_t* __restrict__ sizes, int64_t cap_range) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= F || e >= sizes[kNEntry]) return;    // F: the capacity of the entry buffer
    const FEntry E = ent[e];
    int32_t nr;
    int64_t tot;
    uint64_t m0;
    uint32_t m1;
    entry_ranges<true>(bd, tvs, nodes, E, e, bbox, bboxid, leaf_begin, leaf_count, lmask, rbeg, rpre,
                       rcode, mono, roff_e[e], soff_e[e] - soff_e[eoff[E.blk]], cap_range, nr, tot, m0, m1);
}

// The chunk of a box: the requested one, or larger when the item partial sums (3 x 64
// floats per item) would pass max_items items.  With `adapt` a small box gets
// a smaller one of its own (see kSmallBox), bounded by what the whole batch lists.
struct ChunkArgs {
    const int64_t* soff_e;
    const int64_t* eoff;
    const int64_t* coff;
    const int64_t* choff;
    int64_t chunk_req, max_items;
    int adapt;
};
__device__ int64_t box_chunk_of(const ChunkArgs& A, const int64_t* __restrict__ sizes, int x) {
    const int64_t total = A.soff_e[sizes[kNEntry]];
    int64_t chunk = A.chunk_req;
    const int64_t need = (total + A.max_items - 1) / A.max_items;
    if (need > chunk) chunk = ((need + kBlock - 1) / kBlock) * kBlock;
    if (chunk > INT32_MAX / 2) chunk = INT32_MAX / 2;
    if (A.adapt) {
        const int64_t nblock = sizes[kNBlock];
        const int64_t b0 = A.coff[A.choff[x]], b1 = A.coff[A.choff[x + 1]];
        const int64_t own = A.soff_e[A.eoff[b1 < nblock ? b1 : nblock]] - A.soff_e[A.eoff[b0 < nblock ? b0 : nblock]];
        if (own < kSmallBox) {
            const double root = cbrt((double)own);
            int64_t few = (int64_t)(kChunkScale * root * root / kBlock + 0.5) * kBlock;
            const int64_t floor_ = own < kTinyBox ? kTinyChunk : kSmallChunk;
            if (few < floor_) few = floor_;
            const int64_t least = (total + kEnoughItems * kBlock - 1) / (kEnoughItems * kBlock) * kBlock;
            if (few < least) few = least;
            chunk = few < chunk ? few : chunk;
        }
    }
    return chunk;
}

// The active lanes of every target block, one wave per block.
__global__ void __launch_bounds__(256) block_active_kernel(const int64_t* __restrict__ sizes,
                                                           const uint8_t* __restrict__ active,
                                                           const int32_t* __restrict__ perm,
                                                           const int32_t* __restrict__ bstart,
                                                           const int32_t* __restrict__ bcount,
                                                           uint64_t* __restrict__ bact) {
    const int lane = threadIdx.x & (kBlock - 1);
    const int64_t b = (int64_t)blockIdx.x * (256 / kBlock) + threadIdx.x / kBlock;
    if (b >= sizes[kNBlock]) return;
    const bool on = lane < bcount[b] && active[perm[(int64_t)bstart[b] + lane]] != 0;
    const uint64_t m = __ballot(on);
    if (lane == 0) bact[b] = m;
}

// What the item kernels read and write.
struct ItemBuild {
    ChunkArgs A;
    const int32_t* slen;
    const int32_t* bcount;
    const int32_t* bboxid;
    const uint64_t* bact;        // active lanes per block, or null
    int64_t cap_block, cap_range, cap_item;
    int npass, stop;
    const int64_t* roff;
    const int* bad;
    int64_t* host;               // the host's page-locked copy of the sizes, or null
    int64_t* sizes;
    int32_t* box_chunk;
    int32_t* icount;
    int64_t* ioff;
    int32_t* iblock;
    int32_t* is0;
    int32_t* is1;
};

// Work items of block b: its list in chunks (at least one item, so that every
// target is written); none for a block without an active target when flags
// are given.  With fresh lists (A.soff_e set) the boxes' chunks are found here
// too.  cand: the block's (target, listed source) pairs; the kernel prunes some
// sources further.
__device__ __forceinline__ int32_t block_items(const ItemBuild& I, int64_t b, int64_t& chunk,
                                               unsigned long long& cand) {
    const int x = I.bboxid[b];
    chunk = I.A.soff_e ? box_chunk_of(I.A, I.sizes, x) : I.box_chunk[x];
    if (I.A.soff_e) {
        if (b == 0) I.sizes[kTotalSrc] = I.A.soff_e[I.sizes[kNEntry]];
        if (b == 0 || I.bboxid[b - 1] != x) I.box_chunk[x] = (int32_t)chunk;
    }
    cand = 0;
    if (I.bact && I.bact[b] == 0) return 0;
    const int32_t s = I.slen[b];
    cand = (unsigned long long)s * (unsigned long long)I.bcount[b];
    return s <= 0 ? 1 : (int32_t)((s + chunk - 1) / chunk);
}

// The item and range totals, and the flag that makes the PP kernels return.
__device__ __forceinline__ void finish_items(const ItemBuild& I, int64_t ni) {
    int64_t* sizes = I.sizes;
    const int64_t nr = I.roff[sizes[kNBlock]];
    sizes[kNeedItem] = ni;
    sizes[kNeedRange] = nr;
    sizes[kNItem] = ni < I.cap_item ? ni : I.cap_item;
    sizes[kNRange] = nr < I.cap_range ? nr : I.cap_range;
    if (ni > I.cap_item) sizes[kOverflow] |= 8;
    if (nr > I.cap_range) sizes[kOverflow] |= 4;
    if (sizes[kStart] - I.npass > I.stop) sizes[kOverflow] |= 128;
    if (sizes[kRerun]) sizes[kOverflow] |= 256;
    sizes[kBad] = *I.bad;
    sizes[kSkip] = (sizes[kOverflow] != 0 || sizes[kBad] != 0 || sizes[kMoved] != 0) ? 1 : 0;
}

__device__ __forceinline__ void put_items(const ItemBuild& I, int64_t b, int64_t o, int32_t count, int64_t chunk) {
    const int64_t len = I.slen[b];
    for (int32_t c = 0; c < count; ++c) {
        if (o + c >= I.cap_item) return;
        I.iblock[o + c] = (int32_t)b;
        I.is0[o + c] = (int32_t)(c * chunk);
        I.is1[o + c] = (int32_t)((c + 1) * chunk < len ? (c + 1) * chunk : len);
    }
}

__global__ void item_count_kernel(ItemBuild I) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= I.cap_block) return;
    if (b >= I.sizes[kNBlock]) {
        I.icount[b] = 0;
        return;
    }
    int64_t chunk;
    unsigned long long cand;
    I.icount[b] = block_items(I, b, chunk, cand);
    atomicAdd(reinterpret_cast<unsigned long long*>(I.sizes + kCand), cand);
}

// Writes the items; the first workgroup also finishes the sizes and copies
// them to the host's copy, which saves a copy operation behind the PP kernels.
__global__ void item_fill_kernel(ItemBuild I) {
    int64_t* sizes = I.sizes;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) finish_items(I, I.ioff[sizes[kNBlock]]);
        __threadfence_block();
        __syncthreads();
        if (I.host && threadIdx.x < kSizeSlots) I.host[threadIdx.x] = sizes[threadIdx.x];
    }
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= sizes[kNBlock]) return;
    put_items(I, b, I.ioff[b], I.icount[b], I.box_chunk[I.bboxid[b]]);
}

// Up to kFewItemBlocks blocks: one workgroup counts, scans and writes, a block per
// thread, in the place of three launches (32 k particles: 20 us of kernels and
// two gaps became 16; 1 k: 13 became 8).  Summing the entries here as well took
// as long as the launch it saves: one workgroup waits for its binary searches.
constexpr int kFewItemBlocks = 1024;

__global__ void __launch_bounds__(kFewItemBlocks) item_small_kernel(ItemBuild I) {
    __shared__ int32_t s_wave[kFewItemBlocks / 64];
    __shared__ unsigned long long s_cand;
    int64_t* sizes = I.sizes;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t b = threadIdx.x, nblock = sizes[kNBlock];
    const bool any = b < nblock;
    if (b == 0) s_cand = 0;
    __syncthreads();
    int64_t chunk = 1;
    unsigned long long cand = 0;
    const int32_t n = any ? block_items(I, b, chunk, cand) : 0;
    int32_t upto = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t below = __shfl_up(upto, d);
        cand += __shfl_xor(cand, d);
        if (lane >= d) upto += below;
    }
    if (lane == 63) s_wave[wv] = upto;
    if (lane == 0) atomicAdd(&s_cand, cand);
    __syncthreads();
    int64_t o = upto - n, total = 0;
    for (int k = 0; k < kFewItemBlocks / 64; ++k) {
        if (k == wv) o += total;
        total += s_wave[k];
    }
    if (b < I.cap_block) {
        I.icount[b] = n;
        I.ioff[b] = o;
    }
    if (b == 0) {
        I.ioff[I.cap_block] = total;
        sizes[kCand] += s_cand;
        finish_items(I, total);
    }
    __threadfence_block();
    __syncthreads();
    if (I.host && threadIdx.x < kSizeSlots) I.host[threadIdx.x] = sizes[threadIdx.x];
    if (any) put_items(I, b, o, n, chunk);
}

// Per-pass slots of a pass that reuses the lists (the list counts stay; the
// overflow bits of the last pass go, since the lists' own buffers fitted).
__global__ void zero_sizes_reuse_kernel(int64_t* __restrict__ sizes, int* __restrict__ bad,
                                        int32_t* __restrict__ mass_flag, int nbox) {
    for (int x = threadIdx.x; x < nbox; x += blockDim.x) mass_flag[x] = 0;
    if (threadIdx.x != 0) return;
    sizes[kOverflow] = 0;
    sizes[kCand] = 0;
    sizes[kMoved] = 0;
    sizes[kSkip] = 0;
    sizes[kBad] = 0;
    *bad = 0;
}

// ... and the per-box flags of unequal masses (mass_flag, when given).
__global__ void zero_sizes_kernel(int64_t* __restrict__ sizes, int* __restrict__ bad,
                                  int32_t* __restrict__ mass_flag, int nbox) {
    if (threadIdx.x < kSizeSlots) sizes[threadIdx.x] = 0;
    if (threadIdx.x == 0) *bad = 0;
    if (mass_flag)
        for (int x = threadIdx.x; x < nbox; x += blockDim.x) mass_flag[x] = 0;
}

}  // namespace

// A grid for a grid-stride loop over at most n items.
static unsigned stride_grid(int64_t n, int t) {
    const int64_t b = (n + t - 1) / t;
    return (unsigned)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

// Nodes of the implicit trees over at most n leaves in nbox boxes: the
// leaves plus at most n / 7 + 1 nodes per level above them in every box.
static int64_t tree_node_bound(int64_t n, int nbox) {
    const int64_t m = n > 0 ? n : 1;
    return m + m / 7 + (int64_t)nbox * kTreeMaxLevels + 8;
}

// start_level on the host.
static int host_start_level(int64_t c, int64_t most) {
    int h = 0;
    while (c > 1 && (h == 0 || c > most)) {
        c = (c + 7) / 8;
        ++h;
    }
    return h;
}

static int make_items(const ChunkArgs& chunks, Work& w, hipStream_t s, const uint8_t* active);

// Levels of the implicit tree over at most n leaves.
static int levels_for(int64_t n) {
    int h = 1;
    int64_t c = n > 0 ? n : 1;
    while (c > 1 && h < kTreeMaxLevels) {
        c = (c + 7) / 8;
        ++h;
    }
    return h;
}

// Clears the count slots and the bad-input flag.
int reset_sizes(int nbox, Work& w, hipStream_t s) {
    PP_TRY(w.mass_flag.reserve(sizeof(int32_t) * (nbox + 1)));
    PP_TRY(w.sizes.reserve(sizeof(int64_t) * kSizeSlots));
    PP_TRY(w.bad.reserve(64));
    hipLaunchKernelGGL(zero_sizes_kernel, dim3(1), dim3(kSizeSlots), 0, s, w.sizes.as<int64_t>(),
                       w.bad.as<int>(), w.mass_flag.as<int32_t>(), nbox);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int reset_sizes_reuse(int nbox, Work& w, hipStream_t s) {
    hipLaunchKernelGGL(zero_sizes_reuse_kernel, dim3(1), dim3(64), 0, s, w.sizes.as<int64_t>(),
                       w.bad.as<int>(), w.mass_flag.as<int32_t>(), nbox);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

// Nodes of the start level of the list expansion at most.  Small boxes start
// as low as they can: each level skipped is three launches.  Large ones start
// where a wave tests all nodes at once: the levels below cost less per entry
// than testing every node for every block (2.1 M particles: 316 us from a
// level of 540 nodes, 88 from one of 9).
// chunks up to which the one-launch forms of the block split and of the first
// expansion pass are taken, and room for blocks beyond which that pass takes a
// lane for each
constexpr int64_t kFewChunks = 4096;
constexpr int64_t kManyBlocks = 65536;
static bool small_boxes(int64_t N, int nbox) { return N / nbox <= 131072; }
static int64_t start_nodes_for(int64_t N, int nbox) { return small_boxes(N, nbox) ? 1024 : 128; }

int stage_leaves(const BatchDev& bd, int64_t N, const uint64_t* sorted_keys, Work& w, hipStream_t s) {
    const int nbox = bd.nbox;
    const int64_t m = N > 0 ? N : 1;        // leaves: at most one per particle
    PP_TRY(w.sizes.reserve(sizeof(int64_t) * kSizeSlots));
    PP_TRY(w.loff_dev.reserve(sizeof(int64_t) * (nbox + 1)));
    PP_TRY(w.lbegin.reserve(sizeof(int64_t) * (m + 1)));
    PP_TRY(w.lcount.reserve(sizeof(int32_t) * (m + 1)));
    PP_TRY(w.llevel.reserve(sizeof(int32_t) * (m + 1)));
    PP_TRY(w.lprefix.reserve(sizeof(uint64_t) * (m + 1)));
    PP_TRY(w.tviews.reserve(sizeof(TreeView) * nbox));
    PP_TRY(w.lvl_prefix.reserve(sizeof(int64_t) * (size_t)kTreeMaxLevels * (nbox + 1)));
    PP_TRY(w.group_prefix.reserve(sizeof(int64_t) * (nbox + 1)));
    if (N == 0) {
        hipLaunchKernelGGL(no_leaves_kernel, dim3(1), dim3(64), 0, s, nbox, w.loff_dev.as<int64_t>(),
                           w.sizes.as<int64_t>(), start_nodes_for(N, nbox), w.tviews.as<TreeView>(),
                           w.lvl_prefix.as<int64_t>(), w.group_prefix.as<int64_t>());
        PP_HIP(hipGetLastError());
        return PP_OK;
    }
    // short tiles while there are few of them
    constexpr int kShort = 2, kLong = 8;
    const int ipt = N <= 131072 ? kShort : kLong;
    const int64_t nt = (N + 256 * ipt - 1) / (256 * ipt);
    // a small box's workspace for the whole list builder at once: it is cleared
    // whenever it grows
    if (N <= (1 << 20)) PP_TRY(grow_scan(w.scan_ws, 10 * N + 40960, s));
    PP_TRY(grow_lookback(w.scan_ws, nt, s));
    LbArgs lb;
    PP_TRY(lookback_args(w.scan_ws, nt, &lb));
    auto kernel = ipt == kShort ? leaves_kernel<kShort> : leaves_kernel<kLong>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)nt), dim3(256), 0, s, bd, sorted_keys, N, lb, nt,
                       w.lbegin.as<int64_t>(), w.llevel.as<int32_t>(), w.lprefix.as<uint64_t>(),
                       w.loff_dev.as<int64_t>(), w.sizes.as<int64_t>(), start_nodes_for(N, nbox), w.tviews.as<TreeView>(),
                       w.lvl_prefix.as<int64_t>(), w.group_prefix.as<int64_t>());
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int leaves_to_host(const BatchDev& bd, Work& w, hipStream_t s) {
    w.loff.assign(bd.nbox + 1, 0);
    PP_HIP(hipMemcpyAsync(w.loff.data(), w.loff_dev.p, sizeof(int64_t) * (bd.nbox + 1),
                          hipMemcpyDeviceToHost, s));
    PP_HIP(hipStreamSynchronize(s));
    w.nleaf = w.loff[bd.nbox];
    return PP_OK;
}

int stage_trees(const BatchDev& bd, int64_t N, const double* pos_s, Work& w, hipStream_t s) {
    const int nbox = bd.nbox;
    const int H = levels_for(N);
    w.max_levels = H;
    PP_TRY(w.tree_boxes.reserve(sizeof(IBox) * tree_node_bound(N, nbox)));
    if (nbox > 1) {                              // (the leaves' kernel does it for one box)
        hipLaunchKernelGGL(tree_views_kernel, dim3(1), dim3(256), 0, s, w.loff_dev.as<int64_t>(), nbox,
                           w.tviews.as<TreeView>(), w.lvl_prefix.as<int64_t>(), w.group_prefix.as<int64_t>(),
                           start_nodes_for(N, nbox), w.sizes.as<int64_t>());
        PP_HIP(hipGetLastError());
    }
    if (N == 0) return PP_OK;
    IBox* nodes = w.tree_boxes.as<IBox>();
    const int64_t groups = N / kTreeGroup + nbox;    // bound: leaves may be as many as the particles
    hipLaunchKernelGGL(leaf_tree_kernel, dim3((unsigned)groups), dim3(kTreeGroup), 0, s, bd, pos_s, N,
                       w.tviews.as<TreeView>(), w.group_prefix.as<int64_t>(), w.lbegin.as<int64_t>(),
                       w.sizes.as<int64_t>(), w.lcount.as<int32_t>(), nodes);
    if (H > 4)
        hipLaunchKernelGGL(tree_top_kernel, dim3((unsigned)nbox), dim3(256), 0, s, w.tviews.as<TreeView>(), nodes);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int trees_to_host(const BatchDev& bd, Work& w, hipStream_t s) {
    w.tv.assign(bd.nbox, TreeView{});
    PP_HIP(hipMemcpyAsync(w.tv.data(), w.tviews.p, sizeof(TreeView) * bd.nbox, hipMemcpyDeviceToHost, s));
    PP_HIP(hipStreamSynchronize(s));
    return PP_OK;
}

int stage_node_moments(const BatchDev& bd, int64_t N, Work& w, hipStream_t s) {
    const int nbox = bd.nbox;
    PP_TRY(w.tree_mc.reserve(sizeof(double4) * tree_node_bound(N, nbox)));
    if (N == 0) return PP_OK;
    double4* mc = w.tree_mc.as<double4>();
    hipLaunchKernelGGL(leaf_moment_kernel, dim3(stride_grid(N, 128)), dim3(128), 0, s,
                       w.pos_s.as<double>(), w.mass_s.as<float>(), w.pos_n, w.lbegin.as<int64_t>(),
                       w.sizes.as<int64_t>(), mc);
    int64_t bound = N;
    for (int h = 1; h < w.max_levels; ++h) {
        bound = (bound + 7) / 8 + nbox;
        hipLaunchKernelGGL(tree_moment_kernel, dim3(stride_grid(bound, 256)), dim3(256), 0, s,
                           w.tviews.as<TreeView>(), w.lvl_prefix.as<int64_t>() + (size_t)h * (nbox + 1),
                           nbox, h, mc);
    }
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int build_canonical_pairs(const BatchDev& bd, const Work& w, int64_t W, int64_t T, DevBuf& row_cnt,
                          DevBuf& row_ptr, DevBuf& src, DevBuf& code, DevBuf& scan_ws,
                          int64_t* nentries, hipStream_t s) {
    (void)bd;
    const int64_t nleaf = w.nleaf;     // host copies: leaves_to_host, trees_to_host
    PP_TRY(row_cnt.reserve(sizeof(int32_t) * (nleaf + 1)));
    PP_TRY(row_ptr.reserve(sizeof(int64_t) * (nleaf + 1)));
    *nentries = 0;
    if (nleaf == 0) {
        PP_TRY(launch_scan_i32_to_i64(row_cnt.as<int32_t>(), row_ptr.as<int64_t>(), 0, scan_ws, s));
        PP_HIP(hipStreamSynchronize(s));
        return PP_OK;
    }
    const TreeView tv = w.tv[0];
    const IBox* nodes = w.tree_boxes.as<IBox>();
    hipLaunchKernelGGL(canon_kernel<false>, dim3(blocks_for(nleaf, 64)), dim3(64), 0, s, tv, nodes,
                       nleaf, W, T, row_cnt.as<int32_t>(), (const int64_t*)nullptr,
                       (int32_t*)nullptr, (uint8_t*)nullptr);
    PP_HIP(hipGetLastError());
    PP_TRY(launch_scan_i32_to_i64(row_cnt.as<int32_t>(), row_ptr.as<int64_t>(), nleaf, scan_ws, s));
    int64_t tot = 0;
    PP_TRY(read_back(row_ptr.as<int64_t>() + nleaf, &tot, s));
    PP_TRY(src.reserve(sizeof(int32_t) * (tot + 1)));
    PP_TRY(code.reserve(sizeof(uint8_t) * (tot + 1)));
    hipLaunchKernelGGL(canon_kernel<true>, dim3(blocks_for(nleaf, 64)), dim3(64), 0, s, tv, nodes,
                       nleaf, W, T, (int32_t*)nullptr, row_ptr.as<int64_t>(), src.as<int32_t>(),
                       code.as<uint8_t>());
    PP_HIP(hipGetLastError());
    *nentries = tot;
    return PP_OK;
}

// Capacities start from estimates and grow to 5/4 of what a pass needed
// whenever a buffer was too small (lists_to_host); the pass then runs again.
// (tight: to the need itself.)
static int64_t grow_cap(int64_t cap, int64_t need, bool tight) {
    if (need <= cap) return cap;
    return tight ? need : need + need / 4 + 1024;
}

// After a pass that fitted: a capacity well above the need comes down to it
// (plus the margin).  The grids and scans of the list builder span the
// capacities, so a first guess far above the need (the entry passes start
// from doublings) would otherwise keep costing time on every call.
static int64_t settle_cap(int64_t cap, int64_t need) {
    const int64_t want = need + need / 4 + 1024;
    return cap > want + want / 2 ? want : cap;
}

int stage_lists(const BatchDev& bd, const std::vector<int64_t>& poff, int chunk_req, bool adapt_chunk,
                Work& w, hipStream_t s, const MonoCfg& mcfg, const uint8_t* active) {
    const int nbox = bd.nbox;
    const int64_t N = poff[nbox];
    int64_t* sizes = w.sizes.as<int64_t>();
    // chunks of kBlock particles inside each box (offsets change only with
    // the box sizes; uploaded synchronously then)
    std::vector<int64_t> choff(nbox + 1, 0);
    for (int x = 0; x < nbox; ++x)
        choff[x + 1] = choff[x] + (poff[x + 1] - poff[x] + kBlock - 1) / kBlock;
    const int64_t nc = choff[nbox];
    w.nchunk = nc;
    PP_TRY(w.choff.reserve(sizeof(int64_t) * (nbox + 1)));
    if (choff != w.choff_h) {
        PP_HIP(hipMemcpy(w.choff.p, choff.data(), sizeof(int64_t) * (nbox + 1), hipMemcpyHostToDevice));
        w.choff_h = choff;
    }
    // capacities: blocks from the chunks, the rest from the last need
    if (w.cap_block < nc + nc / 8 + 64) w.cap_block = nc + nc / 8 + 64;
    const int64_t cb = w.cap_block;
    PP_TRY(w.coff.reserve(sizeof(int64_t) * (nc + 2)));
    PP_TRY(w.bstart.reserve(sizeof(int32_t) * cb));
    PP_TRY(w.bcount.reserve(sizeof(int32_t) * cb));
    PP_TRY(w.bbox.reserve(sizeof(IBox) * cb));
    PP_TRY(w.bboxid.reserve(sizeof(int32_t) * cb));
    PP_TRY(w.slen.reserve(sizeof(int32_t) * cb));
    PP_TRY(w.roff.reserve(sizeof(int64_t) * (cb + 2)));
    PP_TRY(w.icount.reserve(sizeof(int32_t) * (cb + 1)));
    PP_TRY(w.ioff.reserve(sizeof(int64_t) * (cb + 2)));
    PP_TRY(w.eoff.reserve(sizeof(int64_t) * (cb + 2)));
    // lowering passes: from the last call's start level (before the first
    // call, that of a guess at the leaves) to level 1, or to level 2 when
    // level 1 would need too many entries; entries that start one level
    // higher than guessed end at level 2, and a larger miss runs the pass again
    if (w.start_level < 0) {
        const int64_t guess = N / nbox / (bd.leaf_max > 8 ? bd.leaf_max / 4 : 2) + 1;
        w.start_level = host_start_level(guess, start_nodes_for(N, nbox));
    }
    const int stop = w.stop_at_level2 ? kDfsLevel : kDfsLevel - 1;
    const int nlower = w.start_level > stop ? w.start_level - stop : 0;
    const int npass = 1 + nlower;
    w.npass = npass;
    // entry capacities, by the level a pass ends at, for exact and for monopole
    // lists (their first guesses fit uniform and clustered boxes at leaf_max 32)
    w.mono_lists = mcfg.on();
    int64_t* caps = w.cap_ent[w.mono_lists ? 1 : 0];
    auto cap = [&](int p) -> int64_t& { return caps[stop + nlower - p]; };
    const int64_t guess[] = {nc > kFewChunks ? 256 : 160, nc > kFewChunks ? 256 : 160, 64, 32};
    for (int p = 0; p < npass; ++p) {
        const int level = stop + nlower - p;
        if (cap(p) < 1024) {
            // monopole lists keep more, smaller nodes: 1.3 to 1.45 times the
            // entries of exact lists of the same particles, where those are known
            const int64_t exact = w.mono_lists ? w.cap_ent[0][level] / 2 * 3 : 0;
            cap(p) = std::max((level < 4 ? guess[level] : 16) * cb, exact);
        }
    }
    int64_t capcnt = cb;
    for (int p = 0; p < npass; ++p) capcnt = cap(p) > capcnt ? cap(p) : capcnt;
    // the scans' workspace for the largest scan of the pass, reserved before
    // the first one is enqueued
    PP_TRY(grow_scan(w.scan_ws, 2 * (capcnt > nc ? capcnt : nc), s));
    const double* pos_s = w.pos_s.as<double>();
    const BlockOut bout{w.bstart.as<int32_t>(), w.bcount.as<int32_t>(), w.bbox.as<IBox>(), w.bboxid.as<int32_t>(), cb};
    if (nc <= kFewChunks) {
        const int64_t nt = (nc + kSplitWaves - 1) / kSplitWaves;
        LbArgs lb;
        PP_TRY(grow_lookback(w.scan_ws, nt, s));
        PP_TRY(lookback_args(w.scan_ws, nt, &lb));
        hipLaunchKernelGGL(block_split_small_kernel, dim3((unsigned)nt), dim3(kSplitWaves * kBlock), 0, s, bd, pos_s, N,
                           w.choff.as<int64_t>(), nc, lb, nt, w.coff.as<int64_t>(), sizes, bout);
    } else {
        PP_TRY(w.ccount.reserve(sizeof(int32_t) * (nc + 1)));
        PP_TRY(w.cbox.reserve(sizeof(IBox) * nc));
        const unsigned groups = blocks_for(nc, 256 / kBlock);
        hipLaunchKernelGGL(block_split_kernel<false>, dim3(groups), dim3(256), 0, s, bd, pos_s, N,
                           w.choff.as<int64_t>(), nc, w.ccount.as<int32_t>(), (const int64_t*)nullptr,
                           w.cbox.as<IBox>(), bout);
        PP_HIP(hipGetLastError());
        const ScanNote note{(int)kNBlock, (int)kNeedBlock, cb, 1ull, -1};
        PP_TRY(launch_scan_i32_to_i64(w.ccount.as<int32_t>(), w.coff.as<int64_t>(), nc, w.scan_ws, s, sizes, &note));
        hipLaunchKernelGGL(block_split_kernel<true>, dim3(groups), dim3(256), 0, s, bd, pos_s, N,
                           w.choff.as<int64_t>(), nc, w.ccount.as<int32_t>(), w.coff.as<int64_t>(),
                           w.cbox.as<IBox>(), bout);
    }
    PP_HIP(hipGetLastError());
    const TreeView* tvs = w.tviews.as<TreeView>();
    const IBox* nodes = w.tree_boxes.as<IBox>();
    const IBox* bbox = w.bbox.as<IBox>();
    const int32_t* bboxid = w.bboxid.as<int32_t>();
    MonoDev mono{mcfg.theta2, mcfg.alpha, mcfg.mc, nullptr};
    if (mcfg.alpha > 0.0) {
        PP_TRY(w.blk_amin2.reserve(sizeof(double) * (cb + 1)));
        hipLaunchKernelGGL(block_amin_kernel, dim3(blocks_for(cb, 256 / kBlock)), dim3(256), 0, s,
                           w.bstart.as<int32_t>(), w.bcount.as<int32_t>(), w.perm.as<int32_t>(),
                           mcfg.acc_ref, w.pos_n, sizes, w.blk_amin2.as<double>());
        PP_HIP(hipGetLastError());
        mono.amin2 = w.blk_amin2.as<double>();
    }
    // Breadth-first expansion: pass 0 takes the nodes of the start levels,
    // every later pass p lowers the entries above level `stop + nlower - p` by
    // one level (entries of boxes with a lower start level wait in the early,
    // short passes), so that the depth-first walks cover at most 8 (else 64)
    // leaves each.  Entry buffers alternate between two arrays.
    int64_t cap_a = 0, cap_b = 0;
    for (int p = 0; p < npass; ++p) {
        int64_t& c = p % 2 == 0 ? cap_a : cap_b;
        c = cap(p) > c ? cap(p) : c;
    }
    PP_TRY(w.fent_a.reserve(sizeof(FEntry) * (cap_a + 1)));
    PP_TRY(w.fent_b.reserve(sizeof(FEntry) * (cap_b + 1)));
    PP_TRY(w.fcnt.reserve(sizeof(int32_t) * (capcnt + 1)));
    PP_TRY(w.foff.reserve(sizeof(int64_t) * (capcnt + 2)));
    PP_TRY(w.fmask.reserve(sizeof(uint16_t) * (capcnt + 1)));
    const int last0 = npass == 1 ? (int)kNEntry : -1;
    if (small_boxes(N, nbox) && nc <= kFewChunks) {
        const int64_t per = kStartWaves / kStartSplit, nt = (cb + per - 1) / per;
        LbArgs lb;
        PP_TRY(grow_lookback(w.scan_ws, nt, s));
        PP_TRY(lookback_args(w.scan_ws, nt, &lb));
        hipLaunchKernelGGL(start_small_kernel, dim3((unsigned)nt), dim3(kStartWaves * kBlock), 0, s, bd, tvs, nodes,
                           bbox, bboxid, lb, nt, sizes, w.fent_a.as<FEntry>(), cap(0), last0, mono);
    } else {
        const bool many = cb > kManyBlocks;
        const unsigned groups = blocks_for(cb, many ? 256 : 256 / kBlock);
        hipLaunchKernelGGL(many ? start_many_kernel<false> : start_kernel<false>, dim3(groups), dim3(256), 0, s, bd,
                           tvs, nodes, bbox, bboxid, (const int64_t*)sizes, cb, w.fcnt.as<int32_t>(),
                           (const int64_t*)nullptr, (FEntry*)nullptr, (int64_t)0, mono);
        PP_HIP(hipGetLastError());
        const ScanNote note{(int)kEntry0, (int)kNeedEntry0, cap(0), 2ull, last0};
        PP_TRY(launch_scan_i32_to_i64(w.fcnt.as<int32_t>(), w.foff.as<int64_t>(), cb, w.scan_ws, s, sizes, &note));
        hipLaunchKernelGGL(many ? start_many_kernel<true> : start_kernel<true>, dim3(groups), dim3(256), 0, s, bd, tvs,
                           nodes, bbox, bboxid, (const int64_t*)sizes, cb, (int32_t*)nullptr, w.foff.as<int64_t>(),
                           w.fent_a.as<FEntry>(), cap(0), mono);
    }
    PP_HIP(hipGetLastError());
    DevBuf* cur = &w.fent_a;
    DevBuf* nxt = &w.fent_b;
    for (int p = 1; p < npass; ++p) {
        const int target = stop + nlower - p;
        const int64_t cin = cap(p - 1), cout = cap(p);
        hipLaunchKernelGGL(bfs_level_kernel<false>, dim3(blocks_for(cin, 128)), dim3(128), 0, s, bd,
                           tvs, nodes, bbox, bboxid, cur->as<FEntry>(),
                           (const int64_t*)(sizes + kEntry0 + p - 1), cin, target, w.fcnt.as<int32_t>(),
                           (const int64_t*)nullptr, (FEntry*)nullptr, (int64_t)0, mono, w.fmask.as<uint16_t>());
        PP_HIP(hipGetLastError());
        const ScanNote note{(int)(kEntry0 + p), (int)(kNeedEntry0 + p), cout, 2ull,
                            p == npass - 1 ? (int)kNEntry : -1};
        PP_TRY(launch_scan_i32_to_i64(w.fcnt.as<int32_t>(), w.foff.as<int64_t>(), cin, w.scan_ws, s, sizes,
                                      &note));
        hipLaunchKernelGGL(bfs_level_kernel<true>, dim3(blocks_for(cin, 128)), dim3(128), 0, s, bd, tvs,
                           nodes, bbox, bboxid, cur->as<FEntry>(),
                           (const int64_t*)(sizes + kEntry0 + p - 1), cin, target, (int32_t*)nullptr,
                           w.foff.as<int64_t>(), nxt->as<FEntry>(), cout, mono, w.fmask.as<uint16_t>());
        PP_HIP(hipGetLastError());
        DevBuf* t = cur;
        cur = nxt;
        nxt = t;
    }
    const int64_t F = cap(npass - 1);          // the final entry buffer's capacity
    const FEntry* ent = cur->as<FEntry>();
    w.ent_final = ent;
    PP_TRY(w.lmask_e.reserve(sizeof(uint64_t) * (F + 1)));
    PP_TRY(w.rcnt_e.reserve(sizeof(int32_t) * (F + 1)));
    PP_TRY(w.scnt_e.reserve(sizeof(int32_t) * (F + 1)));
    PP_TRY(w.roff_e.reserve(sizeof(int64_t) * (F + 2)));
    PP_TRY(w.soff_e.reserve(sizeof(int64_t) * (F + 2)));
    const int64_t* lbegin = w.lbegin.as<int64_t>();
    const int32_t* lcount = w.lcount.as<int32_t>();
    uint64_t* mono0 = nullptr;
    uint8_t* mono1 = nullptr;
    if (mcfg.on()) {
        PP_TRY(w.mono0_e.reserve(sizeof(uint64_t) * (F + 1)));
        PP_TRY(w.mono1_e.reserve(sizeof(uint8_t) * (F + 1)));
        mono0 = w.mono0_e.as<uint64_t>();
        mono1 = w.mono1_e.as<uint8_t>();
    }
    w.mono0 = mono0;
    w.mono1 = mono1;
    if (w.cap_range < 1024) w.cap_range = (nc > kFewChunks ? 320 : 200) * cb;
    if (w.cap_item < 1024) {
        w.cap_item = 2 * cb;
        // small boxes are cut finer: their items grow as the root of the blocks,
        // those of a batch as far as kEnoughItems (twice that here) and else
        // as the blocks (2 to 4 of 2048 positions each)
        int64_t fine = (int64_t)(1000.0 * sqrt((double)cb * nbox));
        if (nbox > 1) fine = std::min(fine, 5 * cb + 2 * kEnoughItems);
        if (adapt_chunk && fine > w.cap_item && cb < nbox * kSmallBlocks) w.cap_item = fine;
    }
    hipLaunchKernelGGL(ranges_count_kernel, dim3(blocks_for(F, 128)), dim3(128), 0, s, bd, tvs, nodes, ent,
                       F, bbox, bboxid, lbegin, lcount, w.lmask_e.as<uint64_t>(), w.rcnt_e.as<int32_t>(),
                       w.scnt_e.as<int32_t>(), mono, mono0, mono1, (const int64_t*)sizes);
    PP_HIP(hipGetLastError());
    PP_TRY(launch_scan2_i32_to_i64(w.rcnt_e.as<int32_t>(), w.scnt_e.as<int32_t>(), w.roff_e.as<int64_t>(),
                                   w.soff_e.as<int64_t>(), F, w.scan_ws, s, sizes));
    hipLaunchKernelGGL(block_sum_kernel, dim3(blocks_for(cb + 1, 256)), dim3(256), 0, s, ent,
                       (const int64_t*)w.roff_e.as<int64_t>(), (const int64_t*)w.soff_e.as<int64_t>(), sizes, cb,
                       w.eoff.as<int64_t>(), w.roff.as<int64_t>(), w.slen.as<int32_t>());
    PP_HIP(hipGetLastError());
    PP_TRY(w.rbeg.reserve(sizeof(int32_t) * (w.cap_range + 1)));
    PP_TRY(w.rpre.reserve(sizeof(int32_t) * (w.cap_range + 1)));
    PP_TRY(w.rcode.reserve(sizeof(uint8_t) * (w.cap_range + 1)));
    hipLaunchKernelGGL(ranges_fill_kernel, dim3(blocks_for(F, 128)), dim3(128), 0, s, bd, tvs, nodes, ent,
                       F, bbox, bboxid, lbegin, lcount, w.lmask_e.as<uint64_t>(),
                       (const int64_t*)w.roff_e.as<int64_t>(), (const int64_t*)w.soff_e.as<int64_t>(),
                       (const int64_t*)w.eoff.as<int64_t>(), w.rbeg.as<int32_t>(), w.rpre.as<int32_t>(),
                       w.rcode.as<uint8_t>(), mono, (const int64_t*)sizes, w.cap_range);
    PP_HIP(hipGetLastError());
    constexpr int64_t kMaxItems = 1 << 21;
    PP_TRY(w.box_chunk.reserve(sizeof(int32_t) * nbox));
    const ChunkArgs chunks{w.soff_e.as<int64_t>(), w.eoff.as<int64_t>(), w.coff.as<int64_t>(),
                           w.choff.as<int64_t>(), chunk_req, kMaxItems, adapt_chunk ? 1 : 0};
    return make_items(chunks, w, s, active);
}

int stage_items(Work& w, hipStream_t s, const uint8_t* active) { return make_items(ChunkArgs{}, w, s, active); }

// The work items; chunks.soff_e null: at the chunks of the current lists.
static int make_items(const ChunkArgs& chunks, Work& w, hipStream_t s, const uint8_t* active) {
    int64_t* sizes = w.sizes.as<int64_t>();
    const int64_t cb = w.cap_block;
    w.active = active;
    if (active) {
        PP_TRY(w.bact.reserve(sizeof(uint64_t) * (cb + 1)));
        hipLaunchKernelGGL(block_active_kernel, dim3(blocks_for(cb, 256 / kBlock)), dim3(256), 0, s, sizes, active,
                           w.perm.as<int32_t>(), w.bstart.as<int32_t>(), w.bcount.as<int32_t>(),
                           w.bact.as<uint64_t>());
    }
    PP_TRY(w.iblock.reserve(sizeof(int32_t) * (w.cap_item + 1)));
    PP_TRY(w.is0.reserve(sizeof(int32_t) * (w.cap_item + 1)));
    PP_TRY(w.is1.reserve(sizeof(int32_t) * (w.cap_item + 1)));
    PP_TRY(w.sizes_h.reserve(sizeof(int64_t) * kSizeSlots));
    ItemBuild I{};
    I.A = chunks;
    I.slen = w.slen.as<int32_t>();
    I.bcount = w.bcount.as<int32_t>();
    I.bboxid = w.bboxid.as<int32_t>();
    I.bact = active ? w.bact.as<uint64_t>() : nullptr;
    I.cap_block = cb;
    I.cap_range = w.cap_range;
    I.cap_item = w.cap_item;
    I.npass = w.npass - 1;
    I.stop = kDfsLevel;
    I.roff = w.roff.as<int64_t>();
    I.bad = w.bad.as<int>();
    I.host = w.sizes_h.pinned ? w.sizes_h.as<int64_t>() : nullptr;
    I.sizes = sizes;
    I.box_chunk = w.box_chunk.as<int32_t>();
    I.icount = w.icount.as<int32_t>();
    I.ioff = w.ioff.as<int64_t>();
    I.iblock = w.iblock.as<int32_t>();
    I.is0 = w.is0.as<int32_t>();
    I.is1 = w.is1.as<int32_t>();
    if (cb <= kFewItemBlocks) {
        hipLaunchKernelGGL(item_small_kernel, dim3(1), dim3(kFewItemBlocks), 0, s, I);
        PP_HIP(hipGetLastError());
        return PP_OK;
    }
    hipLaunchKernelGGL(item_count_kernel, dim3(blocks_for(cb, 256)), dim3(256), 0, s, I);
    PP_HIP(hipGetLastError());
    PP_TRY(launch_scan_i32_to_i64(I.icount, I.ioff, cb, w.scan_ws, s, sizes));
    hipLaunchKernelGGL(item_fill_kernel, dim3(blocks_for(cb, 256)), dim3(256), 0, s, I);
    PP_HIP(hipGetLastError());
    return PP_OK;
}

int lists_to_host(Work& w, hipStream_t s, bool* regrow, bool* moved) {
    *regrow = false;
    if (moved) *moved = false;
    int64_t* h = w.sizes_h.as<int64_t>();
    // page-locked: the last list kernel wrote them there
    if (!w.sizes_h.pinned) PP_HIP(hipMemcpyAsync(h, w.sizes.p, sizeof(int64_t) * kSizeSlots, hipMemcpyDeviceToHost, s));
    PP_HIP(hipStreamSynchronize(s));
    if (h[kBad]) return fail(PP_EINVAL, "non-finite position or mass");
    if (h[kMoved]) {                    // reused lists no longer cover every pair: rebuild
        if (moved) *moved = true;
        *regrow = true;
        return PP_OK;
    }
    if (h[kOverflow] & 64) return fail(PP_EDEVICE, "the list builder's single-pass scan did not complete");
    if (h[kOverflow] & 256) {           // lists of particles out of order: again, sorted by all key bits
        w.full_sort = true;
        *regrow = true;
        return PP_OK;
    }
    if (h[kOverflow] & 16) return fail(PP_ERANGE, "a target block lists more than 2^31 sources");
    if (h[kOverflow]) {
        w.cap_block = grow_cap(w.cap_block, h[kNeedBlock], w.tight);
        const int stop = w.stop_at_level2 ? kDfsLevel : kDfsLevel - 1;
        int np = w.npass;
        if (!w.stop_at_level2 && h[kNeedEntry0 + np - 1] > kEntryBudget) {
            // the level-1 pass would be too large: stop at level 2 from now on
            w.stop_at_level2 = true;
            np -= 1;
        }
        // A pass whose input was cut short counted only what followed from
        // that part: its need is scaled up by what was cut (at most 4 times),
        // so that one more run is enough (a first call at 16M clustered
        // particles: three runs of the lists, 36 ms, became two, 19).
        double cut = 1.0;
        for (int p = 0; p < np; ++p) {
            int64_t& c = w.cap_ent[w.mono_lists ? 1 : 0][stop + w.npass - 1 - p];
            const int64_t need = (int64_t)((double)h[kNeedEntry0 + p] * cut);
            if (need > c && !w.tight) cut = std::min(4.0, std::max(cut, (double)need / (double)c));
            c = grow_cap(c, need, w.tight);
        }
        w.start_level = (int)h[kStart];
        w.cap_range = grow_cap(w.cap_range, (int64_t)((double)h[kNeedRange] * cut), w.tight);
        w.cap_item = grow_cap(w.cap_item, (int64_t)((double)h[kNeedItem] * cut), w.tight);
        *regrow = true;
        return PP_OK;
    }
    // capacities follow the needs (the buffers keep their size): scans and
    // grids then span little more than the data.  Not after a call that had one
    // expansion pass too few: the next one ends at more entries.
    if ((int)h[kStart] <= w.start_level) {
        const int stop = w.stop_at_level2 ? kDfsLevel : kDfsLevel - 1;
        w.cap_block = settle_cap(w.cap_block, h[kNeedBlock]);
        for (int p = 0; p < w.npass; ++p) {
            int64_t& c = w.cap_ent[w.mono_lists ? 1 : 0][stop + w.npass - 1 - p];
            c = settle_cap(c, h[kNeedEntry0 + p]);
        }
        w.cap_range = settle_cap(w.cap_range, h[kNeedRange]);
        // the item count follows the active flags of each call: only a call
        // over every target brings the item capacity down
        if (!w.active) w.cap_item = settle_cap(w.cap_item, h[kNeedItem]);
    }
    w.start_level = (int)h[kStart];
    w.full_sort = h[kRun] != 0;
    w.nleaf = h[kNLeaf];
    w.nblock = h[kNBlock];
    w.nentry = h[kNEntry];
    w.nrange = h[kNRange];
    w.nitem = h[kNItem];
    w.candidates = h[kCand];
    w.total_src = h[kTotalSrc];
    return PP_OK;
}

}  // namespace pp
