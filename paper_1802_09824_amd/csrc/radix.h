// A stable radix sort of (key, number) records, lowest digit first, digits of
// up to 11 bits: per pass a count of every tile's digits, a prefix over the
// tiles and a scatter.  Used for the mesh cells of the PM force (32-bit keys)
// and for the leading bits of the tree keys (64-bit keys).  Nothing waits for
// another workgroup and no memory has to be cleared first.
#pragma once
#include "pp_internal.h"

namespace pp {
namespace {

constexpr int kSortThreads = 512, kSortWaves = kSortThreads / 64;
constexpr int kDigitBits = 11, kDigits = 1 << kDigitBits;

// A record holds its key in .x and a number below 2^32 in .y.
template <class K> struct SortRec;
template <> struct SortRec<uint32_t> {
    using type = uint2;
    static __device__ __forceinline__ uint2 make(uint32_t k, int64_t i) { return make_uint2(k, (uint32_t)i); }
};
template <> struct SortRec<uint64_t> {
    using type = ulonglong2;
    static __device__ __forceinline__ ulonglong2 make(uint64_t k, int64_t i) {
        return make_ulonglong2(k, (unsigned long long)i);
    }
};

struct Digit {
    int shift, bits;
    template <class K>
    __device__ __forceinline__ uint32_t of(K key) const {
        return (uint32_t)(key >> shift) & ((1u << bits) - 1u);
    }
};

// The tile's digit counts (LDS) to its row of the table.
__device__ __forceinline__ void write_counts(const uint32_t* hist, int bits, uint32_t* __restrict__ counts) {
    __syncthreads();
    uint32_t* row = counts + ((int64_t)blockIdx.x << bits);
    for (int d = threadIdx.x; d < 1 << bits; d += kSortThreads) row[d] = hist[d];
}

// Digit counts of the tiles.  FIRST: of the keys alone, in input order.
template <class K, int ITEMS, bool FIRST>
__global__ void __launch_bounds__(kSortThreads) digit_count_kernel(const K* __restrict__ key,
                                                                   const typename SortRec<K>::type* __restrict__ in,
                                                                   int64_t n, Digit dig,
                                                                   uint32_t* __restrict__ counts) {
    __shared__ uint32_t hist[kDigits];
    for (int d = threadIdx.x; d < 1 << dig.bits; d += kSortThreads) hist[d] = 0;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * (kSortThreads * ITEMS) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t p = first + (int64_t)i * kSortThreads;
        if (p < n) atomicAdd(&hist[dig.of(FIRST ? key[p] : (K)in[p].x)], 1u);
    }
    write_counts(hist, dig.bits, counts);
}

// Per digit (a lane each, 64 per workgroup) the counts of the tiles become
// their exclusive prefix over the tiles, and the digit's total is kept.  The
// 16 waves take a stretch of the tiles each.
__global__ void __launch_bounds__(1024) digit_scan_kernel(uint32_t* __restrict__ counts, int64_t ntile, int bits,
                                                          uint32_t* __restrict__ total) {
    __shared__ uint32_t sum[16][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    uint32_t* col = counts + blockIdx.x * 64 + lane;
    const int64_t t0 = ntile * wv / 16, t1 = ntile * (wv + 1) / 16;
    uint32_t mine = 0;
#pragma unroll 8
    for (int64_t t = t0; t < t1; ++t) mine += col[t << bits];
    sum[wv][lane] = mine;
    __syncthreads();
    uint32_t at = 0;
    for (int k = 0; k < wv; ++k) at += sum[k][lane];
    if (wv == 15) total[blockIdx.x * 64 + lane] = at + mine;
#pragma unroll 8
    for (int64_t t = t0; t < t1; ++t) {
        const uint32_t c = col[t << bits];
        col[t << bits] = at;
        at += c;
    }
}

// One pass: every record to its digit's place.  A wave takes 64 ITEMS
// consecutive entries, 64 at a time; lanes with the same digit find one
// another by a ballot per bit, and the first of them moves the wave's count
// of that digit in LDS.  FIRST: `key` alone is read, entry p has number p.
// Bound by the scattered stores of 8 or 16 bytes.
template <class K, int ITEMS, bool FIRST>
__global__ void __launch_bounds__(kSortThreads) digit_scatter_kernel(const K* __restrict__ key,
                                                                     const typename SortRec<K>::type* __restrict__ in,
                                                                     int64_t n, Digit dig,
                                                                     const uint32_t* __restrict__ counts,
                                                                     const uint32_t* __restrict__ total,
                                                                     typename SortRec<K>::type* __restrict__ out) {
    using Rec = typename SortRec<K>::type;
    __shared__ uint16_t cnt[kSortWaves][kDigits];
    __shared__ uint32_t base[kDigits];
    __shared__ uint32_t wsum[kSortWaves];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int D = 1 << dig.bits;
    const int64_t first = (int64_t)blockIdx.x * (kSortThreads * ITEMS) + wv * 64 * ITEMS + lane;
    Rec v[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int64_t p = first + 64 * i;
        v[i] = SortRec<K>::make(0, 0);
        if (p < n) v[i] = FIRST ? SortRec<K>::make(key[p], p) : in[p];
    }
    uint32_t* z = reinterpret_cast<uint32_t*>(cnt);
    for (int d = threadIdx.x; d < kSortWaves * kDigits / 2; d += kSortThreads) z[d] = 0;
    // the digits' first places: totals of the smaller digits, then of the
    // earlier tiles
    constexpr int PER = kDigits / kSortThreads;
    uint32_t t[PER], sum = 0;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = PER * threadIdx.x + k;
        t[k] = d < D ? total[d] : 0u;
        sum += t[k];
    }
    uint32_t upto = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t below = __shfl_up(upto, o);
        if (lane >= o) upto += below;
    }
    if (lane == 63) wsum[wv] = upto;
    __syncthreads();
    uint32_t at = upto - sum;
    for (int k = 0; k < wv; ++k) at += wsum[k];
    const uint32_t* row = counts + ((int64_t)blockIdx.x << dig.bits);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int d = PER * threadIdx.x + k;
        if (d < D) base[d] = at + row[d];
        at += t[k];
    }
    uint32_t rank[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool on = first + 64 * i < n;
        const uint32_t d = dig.of((K)v[i].x);
        uint64_t same = __ballot(on);
        for (int k = 0; k < dig.bits; ++k) {
            const bool bit = (d >> k) & 1u;
            const uint64_t with = __ballot(bit);
            same &= bit ? with : ~with;
        }
        const int below = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
        const uint32_t c = cnt[wv][d];
        wave_sync();
        if (on && below == 0) cnt[wv][d] = (uint16_t)(c + __popcll(same));
        wave_sync();
        rank[i] = c + below;
    }
    __syncthreads();
    for (int d = threadIdx.x; d < D; d += kSortThreads) {
        uint32_t sofar = 0;
#pragma unroll
        for (int k = 0; k < kSortWaves; ++k) {
            const uint32_t c = cnt[k][d];
            cnt[k][d] = (uint16_t)sofar;
            sofar += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (first + 64 * i >= n) break;
        const uint32_t d = dig.of((K)v[i].x);
        out[base[d] + cnt[wv][d] + rank[i]] = v[i];
    }
}

// One pass from the input (FIRST: the keys, else `in`) to `out`; counts: a row
// of 2^bits (at least 64) per tile, `counted` when they are there already.
template <class K, int ITEMS, bool FIRST>
void launch_digit_pass(const K* key, const typename SortRec<K>::type* in, int64_t n, Digit dig, bool counted,
                       uint32_t* counts, uint32_t* total, typename SortRec<K>::type* out, hipStream_t s) {
    const int64_t ntile = (n + kSortThreads * ITEMS - 1) / (kSortThreads * ITEMS);
    const dim3 tiles((unsigned)ntile), threads(kSortThreads);
    if (!counted)
        hipLaunchKernelGGL((digit_count_kernel<K, ITEMS, FIRST>), tiles, threads, 0, s, key, in, n, dig, counts);
    hipLaunchKernelGGL(digit_scan_kernel, dim3(1u << (dig.bits - 6)), dim3(1024), 0, s, counts, ntile, dig.bits, total);
    hipLaunchKernelGGL((digit_scatter_kernel<K, ITEMS, FIRST>), tiles, threads, 0, s, key, in, n, dig, counts, total,
                       out);
}

}  // namespace
}  // namespace pp
