// The long-range particle-mesh (PM) force of sec. 3.1, on one periodic box:
//   1. cloud-in-cell (CIC) assignment of the masses to an N^3 mesh, without
//      atomics on the mesh: the particles are sorted by the mesh cell that
//      holds them (a stable radix sort, so ties keep the input order); each
//      cell's run is cut at every 64th sorted particle and the 8 corner sums
//      of each piece are formed in order, and every mesh point adds the
//      matching corner sums of the 8 cells around it, cells and pieces in a
//      fixed order; the result does not depend on scheduling;
//   2. real-to-complex FFT (hipFFT, FP64);
//   3. the 3-point difference Green function of sec. 3.1,
//      phi_k = -pi G Delta^2 rho_k / (sin^2(pi l/N) + sin^2(pi m/N) + sin^2(pi n/N)),
//      times the long-range filter exp(-k^2 r_s^2) (the complement of the
//      short-range factor of Eq. equ:split), k = 0 dropped;
//   4. complex-to-real FFT to the mesh potential;
//   5. -grad phi on the mesh by the 4-point central difference;
//   6. linear (CIC) interpolation of the mesh acceleration to the particles,
//      taken in the sorted order (neighbouring threads read neighbouring
//      mesh points) and scattered back to the input order.
// Mesh arrays are x-major: point (i, j, k) at (i N + j) N + k, the layout
// hipFFT's 3-D transforms use with the last axis fastest.
#include <cmath>
#include <new>
#include <string>
#include <vector>

#include <hipfft/hipfft.h>

#include "pp_internal.h"
#include "radix.h"

namespace pp {
namespace {

__global__ void zero_f64_kernel(double* __restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

// Lower mesh corner and the weight of the upper corner per axis.
// A wrapped position that rounds to L itself, or a non-finite one, lands
// on point 0 with weight 0 for its upper neighbour, so every index stays in
// [0, N).
__device__ __forceinline__ void cic_corner(double x, double L, double inv_d, int N, int& i0, double& f) {
    double w = (x - L * floor(x / L)) * inv_d;      // wrap into [0, L), mesh units
    if (!(w >= 0.0 && w < (double)N)) w = 0.0;
    const double c = floor(w);
    f = w - c;
    const int i = (int)c;
    i0 = i < N ? i : N - 1;
}

// ------------------------------------------------------- sort by cell --
// Two passes of radix.h for up to 2^22 cells, where a general sort of 64-bit keys
// takes three of 12-byte pairs and clears its look-back state before each: 72 us
// at 2.1 M particles and 128^3 cells, against 144.  Three passes of 7 bits take 79
// (longer runs of writes, one more pass), tiles of 8192 particles 80.
constexpr int kCellItems = 8;
constexpr int kCellTile = kSortThreads * kCellItems;

// Cell of every particle (the key of the sort) and its upper-corner weights
// and mass as one record (input order); the first pass's digit counts; and
// every cell's run cleared.  One workgroup per tile of the sort; with few tiles
// more of them for the clearing (two tiles alone took 60 us for 128^3 cells).
__global__ void __launch_bounds__(kSortThreads) cic_cell_kernel(const double* __restrict__ pos,
                                                                const float* __restrict__ mass, int64_t n,
                                                                double L, double inv_d, int N, Digit dig,
                                                                uint32_t* __restrict__ key,
                                                                double4* __restrict__ rec_in,
                                                                uint32_t* __restrict__ counts,
                                                                int2* __restrict__ run, int64_t cells) {
    __shared__ uint32_t hist[kDigits];
    for (int d = threadIdx.x; d < 1 << dig.bits; d += kSortThreads) hist[d] = 0;
    for (int64_t c = (int64_t)blockIdx.x * kSortThreads + threadIdx.x; c < cells;
         c += (int64_t)gridDim.x * kSortThreads)
        run[c] = make_int2(0, 0);
    if ((int64_t)blockIdx.x * kCellTile >= n) return;
    __syncthreads();
    const int64_t first = (int64_t)blockIdx.x * kCellTile + threadIdx.x;
#pragma unroll 4
    for (int i = 0; i < kCellItems; ++i) {
        const int64_t p = first + (int64_t)i * kSortThreads;
        if (p >= n) break;
        int ix, iy, iz;
        double fx, fy, fz;
        cic_corner(pos[p], L, inv_d, N, ix, fx);
        cic_corner(pos[n + p], L, inv_d, N, iy, fy);
        cic_corner(pos[2 * n + p], L, inv_d, N, iz, fz);
        const uint32_t c = ((uint32_t)ix * N + iy) * N + iz;
        key[p] = c;
        rec_in[p] = make_double4(fx, fy, fz, (double)mass[p]);
        atomicAdd(&hist[dig.of(c)], 1u);
    }
    write_counts(hist, dig.bits, counts);
}

// --------------------------------------------------------- assignment --
// The corner sums of a cell's particles within one 64-entry window of the
// sorted order.  They are stored by window where the particles start with
// the window (so that a long run has a place for each window), else by cell
// or, when there are fewer particles than cells, by the first particle.
struct PartAt {
    int64_t few;         // min(n, cells): places before the windows' own
    int by_cell;
    __device__ __forceinline__ int64_t of(int64_t cell, int64_t k) const {
        return (k & 63) == 0 ? few + (k >> 6) : (by_cell ? cell : k);
    }
};

// One wave per window of 64 sorted particles: the records in sorted order,
// every occupied cell's run of sorted particles, and the 8 corner sums of
// the window's part of each run, in order: corner (a, b, c) of the
// particles' cell gets m prod (a ? f : 1 - f).  8 lanes share a run, a corner
// each, and read the window's records from LDS.  Bound by the gather of the
// records (32 bytes each from a random line): 70 us at 2.1 M particles, where
// the records' gather, the chunks' offsets and their sums took four kernels
// and 159.
__global__ void __launch_bounds__(256) cic_deposit_kernel(const uint2* __restrict__ sorted,
                                                          const double4* __restrict__ rec_in, int64_t n, PartAt pa,
                                                          int2* __restrict__ run, double4* __restrict__ rec,
                                                          double* __restrict__ part) {
    __shared__ double4 s_rec[4][64];
    __shared__ int s_head[4][65];
    __shared__ uint32_t s_cell[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t k0 = (int64_t)blockIdx.x * 256 + 64 * wv, k = k0 + lane;
    if (k0 >= n) return;
    const bool on = k < n;
    const uint2 kv = on ? sorted[k] : make_uint2(0u, 0u);
    uint32_t prev = __shfl_up(kv.x, 1), next = __shfl_down(kv.x, 1);
    if (lane == 0 && k > 0) prev = sorted[k - 1].x;
    if (lane == 63 && k + 1 < n) next = sorted[k + 1].x;
    const bool first = on && (k == 0 || prev != kv.x), last = on && (k + 1 == n || next != kv.x);
    if (first) run[kv.x].x = (int)k;
    if (last) run[kv.x].y = (int)(k + 1);
    if (on) {
        const double4 r = rec_in[kv.y];
        rec[k] = r;
        s_rec[wv][lane] = r;
        s_cell[wv][lane] = kv.x;
    }
    const bool head = first || (on && lane == 0);
    const uint64_t heads = __ballot(head);
    const int nrun = __popcll(heads);
    if (head) s_head[wv][__builtin_amdgcn_mbcnt_hi((uint32_t)(heads >> 32),
                                                   __builtin_amdgcn_mbcnt_lo((uint32_t)heads, 0u))] = lane;
    if (lane == 0) s_head[wv][nrun] = n - k0 < 64 ? (int)(n - k0) : 64;
    wave_sync();
    const int corner = lane & 7;
    for (int h = lane >> 3; h < nrun; h += 8) {
        const int q0 = s_head[wv][h], q1 = s_head[wv][h + 1];
        double w = 0.0;
        for (int q = q0; q < q1; ++q) {
            const double4 r = s_rec[wv][q];
            w += r.w * (corner & 4 ? r.x : 1.0 - r.x) * (corner & 2 ? r.y : 1.0 - r.y) *
                 (corner & 1 ? r.z : 1.0 - r.z);
        }
        part[8 * pa.of(s_cell[wv][q0], k0 + q0) + corner] = w;
    }
}

// Mesh point (i, j, k) takes corner (a, b, c) of cell (i - a, j - b, k - c)
// (periodic): the CIC assignment seen from the mesh, with the cells and
// their windows in a fixed order.  A lane reads the sums of corners c = 0 and
// 1 of the four cells (i - a, j - b, k) together, 16 bytes each; c = 1 belongs
// to the next point of the row, so a lane takes it from the lane before it
// (the first of a wave or a row reads its own).  Bound by the scattered loads:
// 56 us on a 128^3 mesh with 8 loads of 8 bytes per point, 42 so.
__global__ void __launch_bounds__(256) cic_gather_kernel(const int2* __restrict__ run,
                                                         const double* __restrict__ part, PartAt pa, int N,
                                                         double* __restrict__ rho) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)N * N * N;
    const int lane = threadIdx.x & 63;
    const bool on = e < total;
    const uint32_t p = on ? (uint32_t)e : 0u;
    const int k = (int)(p % (uint32_t)N);
    const int j = (int)((p / (uint32_t)N) % (uint32_t)N);
    const int i = (int)(p / (uint32_t)(N * N));
    uint32_t row[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int ci = q & 2 ? (i == 0 ? N - 1 : i - 1) : i, cj = q & 1 ? (j == 0 ? N - 1 : j - 1) : j;
        row[q] = ((uint32_t)ci * N + cj) * N;
    }
    // sums over the four cells at height kz of their corner pairs
    auto pairs = [&](int kz, double& c0, double& c1) {
        int2 r[4];
        double2 w[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) r[q] = run[row[q] + kz];
        const double2* pair = reinterpret_cast<const double2*>(part);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            w[q] = r[q].x < r[q].y ? pair[4 * pa.of(row[q] + kz, r[q].x) + q] : make_double2(0.0, 0.0);
        c0 = 0.0;
        c1 = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c0 += w[q].x;
            c1 += w[q].y;
            for (int64_t o = ((int64_t)(r[q].x >> 6) + 1) << 6; o < r[q].y; o += 64) {
                const double2 v = pair[4 * pa.of(row[q] + kz, o) + q];
                c0 += v.x;
                c1 += v.y;
            }
        }
    };
    double c0, c1, own, low;
    pairs(k, c0, c1);
    low = __shfl_up(c1, 1);
    if (lane == 0 || k == 0) pairs(k == 0 ? N - 1 : k - 1, own, low);
    if (on) rho[e] = c0 + low;
}

// phi_k = -g_k rho_k e^{-k^2 r_s^2}; scale folds in the density 1/Delta^3
// and the 1/N^3 of the unnormalised inverse FFT.
// sin2: sin^2(pi l / N) for l = 0 .. N - 1 (three sines per point took most
// of the time: 19 us on a 128^3 mesh, 12 with the table).
__global__ void __launch_bounds__(256) green_kernel(hipfftDoubleComplex* __restrict__ rk,
                                                    const double* __restrict__ sin2, int N,
                                                    double L, double G, double rs, double scale) {
    const int nzh = N / 2 + 1;
    const int64_t total = (int64_t)N * N * nzh;
    const double pi = 3.14159265358979323846;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const int kz = (int)((uint32_t)e % (uint32_t)nzh);
        const int ky = (int)(((uint32_t)e / (uint32_t)nzh) % (uint32_t)N);
        const int kx = (int)((uint32_t)e / (uint32_t)(nzh * N));
        if (kx == 0 && ky == 0 && kz == 0) {
            rk[e].x = 0.0;
            rk[e].y = 0.0;
            continue;
        }
        const int lx = kx <= N / 2 ? kx : kx - N;
        const int ly = ky <= N / 2 ? ky : ky - N;
        const double S = sin2[kx] + sin2[ky] + sin2[kz];
        const double d = L / N;
        const double k2 = (2.0 * pi / L) * (2.0 * pi / L) * (double)(lx * lx + ly * ly + kz * kz);
        const double f = -pi * G * d * d / S * exp(-k2 * rs * rs) * scale;
        rk[e].x *= f;
        rk[e].y *= f;
    }
}

// -grad phi by (8 (phi[i+1] - phi[i-1]) - (phi[i+2] - phi[i-2])) / (12 Delta),
// the three components of a point side by side.  Rows have N + 1 points, the
// last one the first again, so that the two upper corners of a cell always
// follow the lower ones.
__global__ void __launch_bounds__(256) gradient_kernel(const double* __restrict__ phi, int N,
                                                       double inv_12d, double* __restrict__ g) {
    const int64_t total = (int64_t)N * N * (N + 1);
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total;
         e += (int64_t)gridDim.x * blockDim.x) {
        const uint32_t row = (uint32_t)(e / (N + 1));
        const int kk = (int)(e - (int64_t)row * (N + 1)), k = kk == N ? 0 : kk;
        const int j = (int)(row % (uint32_t)N);
        const int i = (int)(row / (uint32_t)N);
        auto at = [&](int a, int b, int c) { return phi[((int64_t)a * N + b) * N + c]; };
        auto w = [&](int a) { return a >= N ? a - N : (a < 0 ? a + N : a); };
        g[3 * e] = -(8.0 * (at(w(i + 1), j, k) - at(w(i - 1), j, k)) - (at(w(i + 2), j, k) - at(w(i - 2), j, k))) * inv_12d;
        g[3 * e + 1] = -(8.0 * (at(i, w(j + 1), k) - at(i, w(j - 1), k)) - (at(i, w(j + 2), k) - at(i, w(j - 2), k))) * inv_12d;
        g[3 * e + 2] = -(8.0 * (at(i, j, w(k + 1)) - at(i, j, w(k - 1))) - (at(i, j, w(k + 2)) - at(i, j, w(k - 2)))) * inv_12d;
    }
}

// Linear interpolation of the mesh acceleration, in sorted order (neighbouring
// lanes read neighbouring mesh points).  The result goes to its particle as
// one 16-byte store, and unpack_kernel writes the three arrays: three
// scattered stores of 4 bytes each and 24 loads of 8 bytes from three mesh
// arrays took 165 us at 2.1 M particles, this takes 68 + 9.  Bound by the
// scattered stores and the 192 bytes of mesh per particle through the caches.
__global__ void __launch_bounds__(256) cic_interp_kernel(const uint2* __restrict__ sorted,
                                                         const double4* __restrict__ rec, int64_t n,
                                                         int N, const double* __restrict__ g,
                                                         float4* __restrict__ acc4) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const uint2 kv = sorted[k];
    const int iz = (int)(kv.x % (uint32_t)N);
    const int iy = (int)((kv.x / (uint32_t)N) % (uint32_t)N);
    const int ix = (int)(kv.x / (uint32_t)(N * N));
    const double4 r = rec[k];
    const double fx = r.x, fy = r.y, fz = r.z;
    const int xs[2] = {ix, ix + 1 == N ? 0 : ix + 1}, ys[2] = {iy, iy + 1 == N ? 0 : iy + 1};
    const double wx[2] = {1.0 - fx, fx}, wy[2] = {1.0 - fy, fy}, wz[2] = {1.0 - fz, fz};
    double ax = 0, ay = 0, az = 0;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            double q[6];                     // two points along z
            __builtin_memcpy(q, g + 3 * (((int64_t)xs[a] * N + ys[b]) * (N + 1) + iz), sizeof(q));
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double w = wx[a] * wy[b] * wz[c];
                ax += w * q[3 * c];
                ay += w * q[3 * c + 1];
                az += w * q[3 * c + 2];
            }
        }
    acc4[kv.y] = make_float4((float)ax, (float)ay, (float)az, 0.f);
}

__global__ void __launch_bounds__(256) unpack_kernel(const float4* __restrict__ acc4, int64_t n,
                                                     float* __restrict__ acc) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const float4 a = acc4[p];
    acc[p] = a.x;
    acc[n + p] = a.y;
    acc[2 * n + p] = a.z;
}

const char* fft_text(hipfftResult r) {
    switch (r) {
        case HIPFFT_SUCCESS: return "success";
        case HIPFFT_INVALID_PLAN: return "invalid plan";
        case HIPFFT_ALLOC_FAILED: return "allocation failed";
        case HIPFFT_INVALID_VALUE: return "invalid value";
        case HIPFFT_EXEC_FAILED: return "execution failed";
        case HIPFFT_SETUP_FAILED: return "setup failed";
        case HIPFFT_INVALID_SIZE: return "invalid size";
        default: return "hipFFT error";
    }
}

}  // namespace

int fft_fail(int code, const char* what) {
    return fail(code == HIPFFT_ALLOC_FAILED ? PP_ENOMEM : PP_EDEVICE,
                std::string(what) + " failed: " + fft_text((hipfftResult)code));
}

}  // namespace pp

using namespace pp;

struct pp_pm_plan {
    pp_box_params p{};
    int N = 0;
    hipfftHandle fwd = nullptr, inv = nullptr;
    DevBuf rho;        // FP64 [N^3]: density, then potential (in place of the real field)
    DevBuf rk;         // complex [N][N][N/2+1]
    DevBuf g;          // FP64 [N][N][N + 1][3] mesh acceleration (gradient_kernel)
    DevBuf sin2;       // FP64 [N]: sin^2(pi l / N)
    DevBuf key;        // uint32 [n]: cells, input order
    DevBuf pair_a, pair_b;          // uint2 [n]: (cell, particle), sorted by turns
    DevBuf counts, total;           // digit counts of the sort's tiles, totals
    DevBuf rec_in, rec;             // double4 [n]: upper-corner weights, mass (input, sorted order)
    DevBuf run;                     // int2 [N^3]: each cell's run of sorted particles
    DevBuf part;                    // FP64 [places][8]: corner sums (PartAt)
    ~pp_pm_plan() {
        if (fwd) hipfftDestroy(fwd);
        if (inv) hipfftDestroy(inv);
    }
};

#define PM_FFT(call)                                                   \
    do {                                                               \
        hipfftResult r_ = (call);                                      \
        if (r_ != HIPFFT_SUCCESS) return pp::fft_fail((int)r_, #call); \
    } while (0)

extern "C" {

int pp_pm_plan_create(const pp_box_params* p, int32_t n_mesh, pp_pm_plan** out) {
    if (!out) return fail(PP_EINVAL, "out is NULL");
    *out = nullptr;
    PP_TRY(validate_params(p, false));
    if (n_mesh < 4 || n_mesh > 2048) return fail(PP_EINVAL, "n_mesh must be in 4..2048");
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev == 0) return fail(PP_EDEVICE, "no HIP device");
    // cell numbers are 32-bit; the mesh arrays of more cells exceed the memory
    if ((int64_t)n_mesh * n_mesh * n_mesh > UINT32_MAX) return fail(PP_ENOMEM, "the mesh does not fit the device memory");
    pp_pm_plan* pl = new (std::nothrow) pp_pm_plan;
    if (!pl) return fail(PP_ENOMEM, "host allocation failed");
    pl->p = *p;
    pl->N = n_mesh;
    const int64_t N = n_mesh, cells = N * N * N, half = N * N * (N / 2 + 1);
    int rc = pl->rho.reserve(sizeof(double) * cells);
    if (rc == PP_OK) rc = pl->rk.reserve(sizeof(hipfftDoubleComplex) * half);
    if (rc == PP_OK) rc = pl->g.reserve(sizeof(double) * 3 * N * N * (N + 1));
    if (rc == PP_OK) rc = pl->run.reserve(sizeof(int2) * cells);
    if (rc == PP_OK) rc = pl->sin2.reserve(sizeof(double) * N);
    if (rc == PP_OK) {
        std::vector<double> t(N);
        for (int64_t l = 0; l < N; ++l) {
            const double v = sin(M_PI * (double)(l <= N / 2 ? l : N - l) / (double)N);
            t[l] = v * v;
        }
        if (hipMemcpy(pl->sin2.p, t.data(), sizeof(double) * N, hipMemcpyHostToDevice) != hipSuccess)
            rc = fail(PP_EDEVICE, "upload of the mesh's sines failed");
    }
    if (rc == PP_OK) {
        hipfftResult r = hipfftPlan3d(&pl->fwd, n_mesh, n_mesh, n_mesh, HIPFFT_D2Z);
        if (r == HIPFFT_SUCCESS) r = hipfftPlan3d(&pl->inv, n_mesh, n_mesh, n_mesh, HIPFFT_Z2D);
        if (r != HIPFFT_SUCCESS) rc = pp::fft_fail((int)r, "hipfftPlan3d");
    }
    if (rc != PP_OK) {
        delete pl;
        return rc;
    }
    *out = pl;
    return PP_OK;
}

int pp_pm_accel(pp_pm_plan* pl, const double* pos, const float* mass, int64_t n, float* acc,
                void* stream) {
    if (!pl) return fail(PP_EINVAL, "plan is NULL");
    if (n < 0) return fail(PP_EINVAL, "n must be >= 0");
    if (n > 0 && (!pos || !mass || !acc)) return fail(PP_EINVAL, "NULL buffer");
    hipStream_t s = (hipStream_t)stream;
    const int N = pl->N;
    const int64_t cells = (int64_t)N * N * N;
    const double L = pl->p.L, d = L / N;
    if (n > INT32_MAX) return fail(PP_EINVAL, "n must be below 2^31");
    double* rho = pl->rho.as<double>();
    const uint2* sorted = nullptr;       // (cell, particle) by cell
    if (n > 0) {
        int bits = 6;                    // of the cell number
        while (((int64_t)1 << bits) < cells) ++bits;
        const int npass = (bits + kDigitBits - 1) / kDigitBits;
        const int dbits = (bits + npass - 1) / npass;
        const int64_t ntile = (n + kCellTile - 1) / kCellTile;
        const PartAt pa{n < cells ? n : cells, n > cells};
        PP_TRY(pl->key.reserve(sizeof(uint32_t) * n));
        PP_TRY(pl->pair_a.reserve(sizeof(uint2) * n));
        PP_TRY(pl->pair_b.reserve(sizeof(uint2) * n));
        PP_TRY(pl->counts.reserve((sizeof(uint32_t) * ntile) << dbits));
        PP_TRY(pl->total.reserve(sizeof(uint32_t) << dbits));
        PP_TRY(pl->rec.reserve(sizeof(double4) * n));
        PP_TRY(pl->rec_in.reserve(sizeof(double4) * n));
        PP_TRY(pl->part.reserve(sizeof(double) * 8 * (pa.few + n / 64 + 1)));
        uint32_t* counts = pl->counts.as<uint32_t>();
        uint32_t* total = pl->total.as<uint32_t>();
        int2* run = pl->run.as<int2>();
        const int64_t clearing = (cells + 4 * kSortThreads - 1) / (4 * kSortThreads);
        const int64_t most = clearing < 1024 ? clearing : 1024;
        hipLaunchKernelGGL(cic_cell_kernel, dim3((unsigned)(ntile > most ? ntile : most)), dim3(kSortThreads), 0, s,
                           pos, mass, n, L, 1.0 / d, N, Digit{0, dbits}, pl->key.as<uint32_t>(),
                           pl->rec_in.as<double4>(), counts, run, cells);
        uint2* out = pl->pair_a.as<uint2>();
        for (int pass = 0; pass < npass; ++pass) {
            const Digit dig{pass * dbits, dbits};
            if (pass == 0)
                launch_digit_pass<uint32_t, kCellItems, true>(pl->key.as<uint32_t>(), nullptr, n, dig, true, counts,
                                                              total, out, s);
            else
                launch_digit_pass<uint32_t, kCellItems, false>(nullptr, sorted, n, dig, false, counts, total, out, s);
            PP_HIP(hipGetLastError());
            sorted = out;
            out = pass % 2 == 0 ? pl->pair_b.as<uint2>() : pl->pair_a.as<uint2>();
        }
        hipLaunchKernelGGL(cic_deposit_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, sorted,
                           pl->rec_in.as<double4>(), n, pa, run, pl->rec.as<double4>(), pl->part.as<double>());
        hipLaunchKernelGGL(cic_gather_kernel, dim3(blocks_for(cells, 256)), dim3(256), 0, s, run,
                           pl->part.as<double>(), pa, N, rho);
    } else {
        hipLaunchKernelGGL(zero_f64_kernel, dim3(2048), dim3(256), 0, s, rho, cells);
    }
    PP_HIP(hipGetLastError());
    PM_FFT(hipfftSetStream(pl->fwd, s));
    PM_FFT(hipfftSetStream(pl->inv, s));
    hipfftDoubleComplex* rk = pl->rk.as<hipfftDoubleComplex>();
    PM_FFT(hipfftExecD2Z(pl->fwd, rho, rk));
    const double scale = 1.0 / (d * d * d) / (double)cells;
    hipLaunchKernelGGL(green_kernel, dim3(2048), dim3(256), 0, s, rk, pl->sin2.as<double>(), N, L, pl->p.G, pl->p.rs,
                       scale);
    PP_HIP(hipGetLastError());
    PM_FFT(hipfftExecZ2D(pl->inv, rk, rho));
    double* g = pl->g.as<double>();
    hipLaunchKernelGGL(gradient_kernel, dim3(2048), dim3(256), 0, s, rho, N, 1.0 / (12.0 * d), g);
    if (n > 0) {
        float4* acc4 = pl->rec_in.as<float4>();          // the records in input order are no longer needed
        hipLaunchKernelGGL(cic_interp_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, sorted,
                           pl->rec.as<double4>(), n, N, g, acc4);
        hipLaunchKernelGGL(unpack_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, acc4, n, acc);
    }
    PP_HIP(hipGetLastError());
    return PP_OK;
}

void pp_pm_plan_destroy(pp_pm_plan* pl) { delete pl; }

}  // extern "C"
