// The conventional predictor the wavelet route is compared against (section
// 2.2, first step of the major cycle: a forward FFT of the model image, then
// degridding with an anti-aliasing kernel and a w correction).  Written as a
// type-2 non-uniform FFT in (u, v, w):
//   * the model image is divided by the Fourier transform of the kernel in
//     all three directions, multiplied per w plane by exp(s 2 pi i w_q (n - 1 - c)),
//     zero-padded twofold and transformed (one batched hipFFT over the planes);
//   * every visibility then gathers W x W cells from each of the W planes
//     around it, weighted by the "exponential of semicircle" kernel
//     phi(z) = exp(beta (sqrt(1 - z^2) - 1)) (Barnett, Magland & af Klinteberg
//     2019), the w planes being interpolated like u and v (the improved
//     w-stacking of Ye et al. 2021).
// The result approximates the direct sum over the image pixels to about
// 10^(1 - W).
#include <hip/hip_runtime.h>
#include <hipfft/hipfft.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>

#include "api_internal.h"
#include "chunking.h"
#include "device_math.h"

namespace swv {

namespace {

constexpr int kDgBlock = 256;
constexpr int kQuad = 100;           // Gauss-Legendre nodes of the kernel transform
constexpr int kMaxSupport = 16;
constexpr double kBetaPerW = 2.3;

// Gauss-Legendre nodes and weights on [-1, 1]: Newton's method on P_n, with
// P_n from the three-term recurrence k P_k = (2k - 1) z P_{k-1} - (k - 1) P_{k-2}
// and P_n' = n (z P_n - P_{n-1}) / (z^2 - 1); weights 2 / ((1 - z^2) P_n'^2).
void gauss_legendre(int n, double* x, double* wt) {
    for (int i = 0; i < (n + 1) / 2; ++i) {
        double z = std::cos(M_PI * (i + 0.75) / (n + 0.5));
        double pn = 0, dpn = 1;
        for (int it = 0; it < 12; ++it) {
            double p0 = 1.0, p1 = z;
            for (int k = 2; k <= n; ++k) {
                const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
                p0 = p1;
                p1 = p2;
            }
            pn = p1;
            dpn = n * (z * p1 - p0) / (z * z - 1.0);
            z -= pn / dpn;
        }
        double p0 = 1.0, p1 = z;
        for (int k = 2; k <= n; ++k) {
            const double p2 = ((2.0 * k - 1.0) * z * p1 - (k - 1.0) * p0) / k;
            p0 = p1;
            p1 = p2;
        }
        dpn = n * (z * p1 - p0) / (z * z - 1.0);
        x[i] = -z;
        x[n - 1 - i] = z;
        wt[i] = wt[n - 1 - i] = 2.0 / ((1.0 - z * z) * dpn * dpn);
    }
}

__host__ __device__ __forceinline__ double es_phi(double z, double beta) {
    const double t = 1.0 - z * z;
    return t >= 0.0 ? exp(beta * (sqrt(t) - 1.0)) : 0.0;
}

// phi_hat(f) = sum_k coef_k cos(2 pi f x_k): Gauss-Legendre in theta with
// x = (W / 2) sin(theta), coef_k = exp(beta (cos theta_k - 1)) cos theta_k w_k (pi / 2) (W / 2)
struct Quadrature {
    double x[kQuad], coef[kQuad];
};

__device__ __forceinline__ double cos_turns(double t) {
    double c, q4;
    cis2pi_q(t - rint(t), c, q4);
    return c;
}

__device__ double es_hat(double f, const Quadrature& q) {
    double s = 0.0;
    for (int k = 0; k < kQuad; ++k) s = fma(q.coef[k], cos_turns(f * q.x[k]), s);
    return s;
}

// Kernel transforms of both image axes: h[i] at offset (i - nx / 2) / Nx for i <
// nx, then those of y.  A wave per value: the few hundred of them are bound by
// the length of a thread's chain.
__global__ __launch_bounds__(kDgBlock) void k_hat_1d(int nx, int ny, int Nx, int Ny, Quadrature q,
                                                     double* __restrict__ h) {
    const int i = (int)(blockIdx.x * (kDgBlock / 64) + (threadIdx.x >> 6));
    if (i >= nx + ny) return;
    const double f = i < nx ? (double)(i - nx / 2) / Nx : (double)(i - nx - ny / 2) / Ny;
    double s = 0.0;
    for (int k = threadIdx.x & 63; k < kQuad; k += 64)
        s = fma(q.coef[k], cos_turns(f * q.x[k]), s);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) h[i] = s;
}

// base[p] = I[p] / (hy hx hw), sn[p] = n_p - 1 - c
__global__ __launch_bounds__(kDgBlock) void k_degrid_prep(
    int nx, int ny, double cell, double c, double dw, const double* __restrict__ image,
    const double* __restrict__ hx, const double* __restrict__ hy, Quadrature quad,
    double* __restrict__ base, double* __restrict__ sn) {
    const int64_t p = (int64_t)blockIdx.x * kDgBlock + threadIdx.x;
    if (p >= (int64_t)nx * ny) return;
    const int iy = (int)(p / nx), ix = (int)(p - (int64_t)iy * nx);
    const double l = (double)(ix - nx / 2) * cell, m = (double)(iy - ny / 2) * cell;
    const double r2 = l * l + m * m;
    const double s = -r2 / (1.0 + sqrt(1.0 - r2)) - c;
    const double hw = es_hat(dw * s, quad);
    base[p] = image[p] / (hy[iy] * hx[ix] * hw);
    sn[p] = s;
}

// Plane q, padded cell (ky, kx): the image pixel at offset t = k (k below the
// image's positive half) or t = k - N (the wrapped negative half), else 0.
__global__ __launch_bounds__(kDgBlock) void k_fill_planes(
    int nx, int ny, int Nx, int Ny, int64_t n_planes, double w0, double dw, int sign,
    const double* __restrict__ base, const double* __restrict__ sn, double2* __restrict__ G) {
    const int64_t cells = (int64_t)Nx * Ny;
    const int64_t i = (int64_t)blockIdx.x * kDgBlock + threadIdx.x;
    if (i >= n_planes * cells) return;
    const int64_t q = i / cells;
    const int64_t r = i - q * cells;
    const int ky = (int)(r / Nx), kx = (int)(r - (int64_t)ky * Nx);
    const int cx = nx / 2, cy = ny / 2;
    int ty = ky <= ny - 1 - cy ? ky : (ky >= Ny - cy ? ky - Ny : INT_MIN);
    int tx = kx <= nx - 1 - cx ? kx : (kx >= Nx - cx ? kx - Nx : INT_MIN);
    double2 out = make_double2(0.0, 0.0);
    if (ty != INT_MIN && tx != INT_MIN) {
        const int64_t p = (int64_t)(ty + cy) * nx + (tx + cx);
        const double wq = w0 + (double)q * dw;
        const double t = wq * sn[p];
        double cs, q4;
        cis2pi_q(t - rint(t), cs, q4);
        const double b = base[p];
        out = make_double2(b * cs, b * (sign * 4.0 * q4));
    }
    G[i] = out;
}

// A group of LV lanes per visibility (4, 8 or 16, the least that holds W): lane a
// takes cell ceil(x - W/2) + a of every grid row, so a row of the stencil is one
// contiguous read of the group, and the 3 W kernel weights are one exponential
// per lane and direction.  With a visibility per lane every 16-byte cell was a
// cache line of its own, and each lane computed all 3 W weights.  707,616 rows,
// W = 10: 3.5 -> 0.93 ms, half of the lines from L1 and the rest at about 20 TB/s
// from L2, which bound it; rows sorted by tile, 0.60 ms, 19 TB/s of cells (L1
// gives a line per clock and CU: 0.46 ms).  Handing each XCD a contiguous run of
// unsorted rows took 1.16 ms.
//
// Rows in records (rows != null) are read from there and say where their
// visibility goes; otherwise row j is the j-th of u, v, w.
//
// Cell W of a direction lies outside the support unless x - W/2 is an integer,
// and then takes weight phi(+-1) like the first; it is a rare extra step.
__device__ __forceinline__ int wrap_index(int64_t k, int n) {
    int r;
    if (k == (int64_t)(int)k)
        r = (int)k % n;
    else
        r = (int)(k % n);
    return r < 0 ? r + n : r;
}

// One row and its place.
struct alignas(32) DgRow {
    double u, v, w;
    long long j;
};

template <int W>
__global__ __launch_bounds__(kDgBlock) void k_degrid(
    int64_t n_vis, const DgRow* __restrict__ rows, const double* __restrict__ u, const double* __restrict__ v,
    const double* __restrict__ w, int Nx, int Ny, int64_t n_planes, double cell, double w0,
    double dw, double c, double beta, int sign, const double2* __restrict__ G,
    double2* __restrict__ out) {
    constexpr int LV = W <= 4 ? 4 : (W <= 8 ? 8 : 16);
    const int a = threadIdx.x & (LV - 1);
    int64_t j = (int64_t)blockIdx.x * (kDgBlock / LV) + threadIdx.x / LV;
    if (j >= n_vis) return;   // whole groups
    double uj, vj, wj;
    if (rows) {
        const DgRow r = rows[j];
        uj = r.u;
        vj = r.v;
        wj = r.w;
        j = r.j;
    } else {
        uj = u[j];
        vj = v[j];
        wj = w[j];
    }
    const double h = 0.5 * W;
    const double xi = uj * Nx * cell, zeta = vj * Ny * cell, eta = (wj - w0) / dw;
    // non-finite or absurd coordinates give NaN, never an index
    if (!(fabs(xi) < 0x1p50 && fabs(zeta) < 0x1p50 && eta >= 0.0 && eta <= (double)n_planes)) {
        if (a == 0) out[j] = make_double2(NAN, NAN);
        return;
    }
    const int64_t x0 = (int64_t)ceil(xi - h), y0 = (int64_t)ceil(zeta - h);
    const int64_t q0 = (int64_t)ceil(eta - h);
    // the lane's weights, and those of cell W
    const double fx = a < W ? es_phi((xi - (double)(x0 + a)) / h, beta) : 0.0;
    const double fya = a < W ? es_phi((zeta - (double)(y0 + a)) / h, beta) : 0.0;
    double fqa = 0.0;
    if (a < W && q0 + a >= 0 && q0 + a < n_planes) fqa = es_phi((eta - (double)(q0 + a)) / h, beta);
    const double fxe = es_phi((xi - (double)(x0 + W)) / h, beta);
    const double fye = es_phi((zeta - (double)(y0 + W)) / h, beta);
    const double fqe = q0 + W < n_planes ? es_phi((eta - (double)(q0 + W)) / h, beta) : 0.0;
    double fy[W];
    int row[W + 1];
    int ky = wrap_index(y0, Ny);
#pragma unroll
    for (int b = 0; b <= W; ++b) {
        if (b < W) fy[b] = __shfl(fya, b, LV);
        row[b] = ky * Nx;   // below 2^30
        if (++ky == Ny) ky = 0;
    }
    // sum over planes and rows of one column of cells
    const auto column = [&](int kx, double& sr, double& si) {
        sr = si = 0.0;
#pragma unroll 1
        for (int t = 0; t <= W; ++t) {
            const double fq = t < W ? __shfl(fqa, t, LV) : fqe;
            if (fq == 0.0) continue;
            const double2* P = G + (q0 + t) * ((int64_t)Nx * Ny) + kx;
            double pr = 0.0, pi = 0.0;
#pragma unroll
            for (int b = 0; b < W; ++b) {
                const double2 g = P[row[b]];
                pr = fma(fy[b], g.x, pr);
                pi = fma(fy[b], g.y, pi);
            }
            if (__builtin_expect(fye != 0.0, 0)) {
                const double2 g = P[row[W]];
                pr = fma(fye, g.x, pr);
                pi = fma(fye, g.y, pi);
            }
            sr = fma(fq, pr, sr);
            si = fma(fq, pi, si);
        }
    };
    const int k0 = wrap_index(x0, Nx);
    double vr = 0.0, vi = 0.0;
    if (a < W) {
        column((k0 + a) % Nx, vr, vi);
        vr *= fx;
        vi *= fx;
    }
    if (__builtin_expect(fxe != 0.0, 0)) {   // the same for the whole group
        double er, ei;
        column((k0 + W) % Nx, er, ei);
        if (a == 0) {
            vr = fma(fxe, er, vr);
            vi = fma(fxe, ei, vi);
        }
    }
#pragma unroll
    for (int o = LV / 2; o > 0; o >>= 1) {
        vr += __shfl_xor(vr, o, LV);
        vi += __shfl_xor(vi, o, LV);
    }
    const double t = wj * c;
    double cs, q4;
    cis2pi_q(t - rint(t), cs, q4);
    const double sn = sign * 4.0 * q4;
    if (a == 0) out[j] = make_double2(vr * cs - vi * sn, vr * sn + vi * cs);
}

// Rows put in the order of their tile, so that what is in flight on a CU shares
// cells in L1 (any order within a tile: a row's result depends on itself alone).
// A counting sort: a histogram, its prefix sums, then every workgroup reserves a
// run in each tile that its rows lie in, 0.04 ms for 707,616 rows.  Tiles are 2^shift cells square, the
// least that keeps to kTiles of them.
constexpr int kTiles = 1024;
constexpr int kSortBlock = 512, kSortPer = 4;

struct Tiles {
    int Nx, Ny, shift, across;
    double cell;
};

__device__ __forceinline__ int tile_of(const Tiles& t, double u, double v) {
    const double xi = u * t.Nx * t.cell, zeta = v * t.Ny * t.cell;
    if (!(fabs(xi) < 0x1p50 && fabs(zeta) < 0x1p50)) return 0;
    const int x = wrap_index((int64_t)floor(xi), t.Nx), y = wrap_index((int64_t)floor(zeta), t.Ny);
    return (y >> t.shift) * t.across + (x >> t.shift);
}

__global__ void k_zero_tiles(int* __restrict__ count) {
    count[blockIdx.x * blockDim.x + threadIdx.x] = 0;
}

__global__ __launch_bounds__(kSortBlock) void k_count_tiles(int n, const double* __restrict__ u,
                                                            const double* __restrict__ v, Tiles t,
                                                            int* __restrict__ count) {
    __shared__ int h[kTiles];
    for (int i = threadIdx.x; i < kTiles; i += kSortBlock) h[i] = 0;
    __syncthreads();
    const int i0 = blockIdx.x * (kSortBlock * kSortPer) + threadIdx.x;
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
        const int i = i0 + r * kSortBlock;
        if (i < n) atomicAdd(&h[tile_of(t, u[i], v[i])], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kTiles; i += kSortBlock)
        if (h[i]) atomicAdd(&count[i], h[i]);
}

// Counts to the tiles' first places (exclusive sums), one workgroup.
__global__ __launch_bounds__(kTiles) void k_tile_starts(int* __restrict__ count) {
    __shared__ int s[kTiles / 64];
    const int own = count[threadIdx.x], lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = own;
    for (int o = 1; o < 64; o *= 2) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) s[wave] = x;
    __syncthreads();
    for (int k = 0; k < wave; ++k) x += s[k];
    count[threadIdx.x] = x - own;
}

__global__ __launch_bounds__(kSortBlock) void k_place_rows(
    int n, const double* __restrict__ u, const double* __restrict__ v,
    const double* __restrict__ w, Tiles t, int* __restrict__ next, DgRow* __restrict__ rows) {
    __shared__ int h[kTiles];
    for (int i = threadIdx.x; i < kTiles; i += kSortBlock) h[i] = 0;
    __syncthreads();
    const int i0 = blockIdx.x * (kSortBlock * kSortPer) + threadIdx.x;
    int tile[kSortPer], rank[kSortPer];
    double ur[kSortPer], vr[kSortPer], wr[kSortPer];
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
        const int i = i0 + r * kSortBlock;
        if (i >= n) continue;
        ur[r] = u[i];
        vr[r] = v[i];
        wr[r] = w[i];
        tile[r] = tile_of(t, ur[r], vr[r]);
        rank[r] = atomicAdd(&h[tile[r]], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kTiles; i += kSortBlock)
        if (h[i]) h[i] = atomicAdd(&next[i], h[i]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kSortPer; ++r) {
        const int i = i0 + r * kSortBlock;
        if (i < n) rows[h[tile[r]] + rank[r]] = DgRow{ur[r], vr[r], wr[r], (long long)i};
    }
}

// Rows are sorted in slabs of this many (64 MB of records).
constexpr int64_t kSortSlab = int64_t(1) << 21;
constexpr size_t kTileBytes = sizeof(int) * kTiles;

// Whether sorting pays, whole calls unsorted and sorted: 707,616 rows, 256 x 256
// pixels, support 10 (96 MB of planes): 1.08 and 0.75 ms; 100,000 of them 0.299 and
// 0.273, 50,000 0.235 and 0.232; 300,000 rows, support 8, 6.4 MB: 0.220 and 0.193.
// Planes that an XCD's 4 MB of L2 hold: 0.327 and 0.350 (support 10, 70 x 70
// pixels); support 6: 0.265 either way.
bool sort_rows(int support, int64_t n_vis, size_t plane_bytes) {
    return support > 6 && n_vis >= 65536 && plane_bytes > (size_t(4) << 20);
}

size_t sort_bytes(int64_t n_vis) {
    return kTileBytes + sizeof(DgRow) * (size_t)std::min(n_vis, kSortSlab);
}

Tiles tiles_of(int Nx, int Ny, double cell) {
    int shift = 0;
    while ((int64_t)(((Nx - 1) >> shift) + 1) * (((Ny - 1) >> shift) + 1) > kTiles) ++shift;
    return Tiles{Nx, Ny, shift, ((Nx - 1) >> shift) + 1, cell};
}

template <int W>
void launch_degrid_w(hipStream_t s, int64_t n_vis, const double* u, const double* v,
                     const double* w, int Nx, int Ny, int64_t nq, double cell, double w0,
                     double dw, double c, double beta, int sign, const double2* G, double2* out,
                     void* sorted) {
    constexpr int LV = W <= 4 ? 4 : (W <= 8 ? 8 : 16);
    const Tiles t = tiles_of(Nx, Ny, cell);
    int* next = (int*)sorted;
    DgRow* rows = sorted ? (DgRow*)((char*)sorted + kTileBytes) : nullptr;
    // rows in slabs that stay within a launch's threads, or the records
    const int64_t slab = sorted ? kSortSlab : kMaxLaunchThreads / LV;
    for (int64_t j = 0; j < n_vis; j += slab) {
        const int64_t n = std::min<int64_t>(slab, n_vis - j);
        if (sorted) {
            constexpr int per = kSortBlock * kSortPer;
            const unsigned nb = (unsigned)((n + per - 1) / per);
            k_zero_tiles<<<kTiles / 256, 256, 0, s>>>(next);
            k_count_tiles<<<nb, kSortBlock, 0, s>>>((int)n, u + j, v + j, t, next);
            k_tile_starts<<<1, kTiles, 0, s>>>(next);
            k_place_rows<<<nb, kSortBlock, 0, s>>>((int)n, u + j, v + j, w + j, t, next, rows);
        }
        k_degrid<W><<<(unsigned)((n * LV + kDgBlock - 1) / kDgBlock), kDgBlock, 0, s>>>(
            n, rows, u + j, v + j, w + j, Nx, Ny, nq, cell, w0, dw, c, beta, sign, G, out + j);
    }
}

using DegridFn = void (*)(hipStream_t, int64_t, const double*, const double*, const double*, int,
                          int, int64_t, double, double, double, double, double, int,
                          const double2*, double2*, void*);
constexpr DegridFn kDegrid[] = {
    nullptr, nullptr, launch_degrid_w<2>, launch_degrid_w<3>, launch_degrid_w<4>,
    launch_degrid_w<5>, launch_degrid_w<6>, launch_degrid_w<7>, launch_degrid_w<8>,
    launch_degrid_w<9>, launch_degrid_w<10>, launch_degrid_w<11>, launch_degrid_w<12>,
    launch_degrid_w<13>, launch_degrid_w<14>, launch_degrid_w<15>, launch_degrid_w<16>};

// w range: kMinmaxBlocks partial (min, max) pairs, then one block combines them.
constexpr int kMinmaxBlocks = 512;

__device__ __forceinline__ void block_minmax(double& lo, double& hi, double* smin,
                                             double* smax) {
    smin[threadIdx.x] = lo;
    smax[threadIdx.x] = hi;
    __syncthreads();
    for (int s = kDgBlock / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + s]);
            smax[threadIdx.x] = fmax(smax[threadIdx.x], smax[threadIdx.x + s]);
        }
        __syncthreads();
    }
    lo = smin[0];
    hi = smax[0];
}

__global__ __launch_bounds__(kDgBlock) void k_minmax_partial(int64_t n,
                                                             const double* __restrict__ x,
                                                             double* __restrict__ part) {
    __shared__ double smin[kDgBlock], smax[kDgBlock];
    double lo = HUGE_VAL, hi = -HUGE_VAL;
    for (int64_t i = (int64_t)blockIdx.x * kDgBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kDgBlock) {
        lo = fmin(lo, x[i]);
        hi = fmax(hi, x[i]);
    }
    block_minmax(lo, hi, smin, smax);
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = lo;
        part[2 * blockIdx.x + 1] = hi;
    }
}

__global__ __launch_bounds__(kDgBlock) void k_minmax_final(int n_part,
                                                           const double* __restrict__ part,
                                                           double* __restrict__ out) {
    __shared__ double smin[kDgBlock], smax[kDgBlock];
    double lo = HUGE_VAL, hi = -HUGE_VAL;
    for (int i = threadIdx.x; i < n_part; i += kDgBlock) {
        lo = fmin(lo, part[2 * i]);
        hi = fmax(hi, part[2 * i + 1]);
    }
    block_minmax(lo, hi, smin, smax);
    if (threadIdx.x == 0) {
        out[0] = lo;
        out[1] = hi;
    }
}

// Nodes and coefficients of es_hat (the Gauss-Legendre rule is made once).
Quadrature quadrature(int support, double beta) {
    static const struct Rule {
        double z[kQuad], wt[kQuad];
        Rule() { gauss_legendre(kQuad, z, wt); }
    } rule;
    Quadrature q;
    for (int k = 0; k < kQuad; ++k) {
        // x = (W / 2) sin(theta), theta = (pi / 2) z: a smooth integrand
        const double th = 0.5 * M_PI * rule.z[k];
        q.x[k] = 0.5 * support * std::sin(th);
        q.coef[k] = std::exp(beta * (std::cos(th) - 1.0)) * std::cos(th) * rule.wt[k] *
                    (0.5 * M_PI) * (0.5 * support);
    }
    return q;
}

unsigned blocks_of(int64_t n) { return (unsigned)((n + kDgBlock - 1) / kDgBlock); }

}  // namespace

void destroy_fft_plan(void* plan) {
    if (plan) (void)hipfftDestroy((hipfftHandle)plan);
}

}  // namespace swv

using namespace swv;

extern "C" int swv_predict_degrid(swv_ctx ctx, int nx, int ny, double cell, const double* image,
                                  int64_t n_vis, const double* u, const double* v,
                                  const double* w, int support, int sign, void* vis_out,
                                  swv_degrid_stats_t* stats) {
    if (!ctx) return fail(SWV_EINVAL, "swv_predict_degrid: null context");
    if (nx < 1 || ny < 1 || nx > 16384 || ny > 16384)
        return fail(SWV_EINVAL, "swv_predict_degrid: grid %d x %d outside 1 .. 16384", nx, ny);
    if (!(cell > 0.0) || !std::isfinite(cell))
        return fail(SWV_EDOMAIN, "swv_predict_degrid: cell must be positive and finite");
    if (support < 2 || support > kMaxSupport)
        return fail(SWV_EINVAL, "swv_predict_degrid: support %d outside 2 .. 16", support);
    if (sign != 1 && sign != -1) return fail(SWV_EDOMAIN, "sign must be +1 or -1 (got %d)", sign);
    if (n_vis < 0) return fail(SWV_EINVAL, "swv_predict_degrid: negative n_vis");
    if (!image || (n_vis > 0 && (!u || !v || !w || !vis_out)))
        return fail(SWV_EINVAL, "swv_predict_degrid: null argument");
    // n - 1 over the grid: 0 at the centre pixel, lowest at the farthest corner
    const int cx = nx / 2, cy = ny / 2;
    double lo = 0.0;
    for (int ix : {0, nx - 1})
        for (int iy : {0, ny - 1}) {
            const double l = (double)(ix - cx) * cell, m = (double)(iy - cy) * cell;
            const double r2 = l * l + m * m;
            if (!(r2 < 1.0)) return fail(SWV_EDOMAIN, "swv_predict_degrid: grid leaves the unit disk");
            lo = std::fmin(lo, -r2 / (1.0 + std::sqrt(1.0 - r2)));
        }
    const double hi = 0.0;
    const double extent = std::fmax(hi - lo, 1e-300);
    const double c = 0.5 * (lo + hi);
    const double dw = 1.0 / (2.0 * extent);
    const int Nx = 2 * nx, Ny = 2 * ny;
    const double beta = kBetaPerW * support;
    if (stats) *stats = swv_degrid_stats_t{};
    if (n_vis == 0) return SWV_OK;
    DeviceGuard guard(ctx->device);
    if (!guard.ok) return fail(SWV_EHIP, "swv_predict_degrid: cannot select device");
    const hipStream_t s = ctx->stream;
    const auto t0 = std::chrono::steady_clock::now();
    // w range of the rows
    int rc = ensure(ctx, ctx->partial2, 16 * (kMinmaxBlocks + 1));
    if (rc) return rc;
    double* d_mm = (double*)ctx->partial2.p;
    const int nb = (int)std::min<int64_t>(kMinmaxBlocks, (n_vis + kDgBlock - 1) / kDgBlock);
    k_minmax_partial<<<nb, kDgBlock, 0, s>>>(n_vis, w, d_mm + 2);
    k_minmax_final<<<1, kDgBlock, 0, s>>>(nb, d_mm + 2, d_mm);
    const Quadrature quad = quadrature(support, beta);   // while the GPU finds the range
    double mm[2];
    hipError_t e = hipMemcpyAsync(mm, d_mm, 16, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(e, "swv_predict_degrid: w range");
    if (!std::isfinite(mm[0]) || !std::isfinite(mm[1]))
        return fail(SWV_EDOMAIN, "swv_predict_degrid: non-finite w");
    const double w0 = mm[0] - 0.5 * support * dw;
    const double nq_f = std::floor((mm[1] - w0) / dw + 0.5 * support) + 1.0;
    const int64_t cells = (int64_t)Nx * Ny;
    if (!(nq_f * (double)cells * 16.0 <= 64.0 * (1ull << 30)))
        return fail(SWV_ENOMEM,
                    "swv_predict_degrid: %.0f w planes of %d x %d cells exceed 64 GiB "
                    "(field too wide for the w range)", nq_f, Nx, Ny);
    const int64_t nq = (int64_t)nq_f;
    // planes go through the FFT a few at a time: a plan for each plane count (it
    // follows the rows' w range) took 8 ms whenever the count changed.  As many
    // planes as keep a transform busy; the last batch may run over the end.
    const int64_t batch = cells >= (1 << 21) ? 1 : cells >= (1 << 20) ? 2 : cells >= (1 << 19) ? 4 : 8;
    const int64_t nq_pad = (nq + batch - 1) / batch * batch;
    // scratch: planes, then base, sn, hx, hy, then the sorted rows
    const int64_t n_pix = (int64_t)nx * ny;
    const size_t plane_bytes = 16 * (size_t)(nq * cells);
    const size_t padded = 16 * (size_t)(nq_pad * cells);
    const size_t extra = (8 * (size_t)(2 * n_pix + nx + ny) + 31) / 32 * 32;
    bool sort = sort_rows(support, n_vis, plane_bytes);
    if (sort && ensure(ctx, ctx->degrid, padded + extra + sort_bytes(n_vis)) != SWV_OK)
        sort = false;   // no room for the records: rows as they come
    rc = sort ? SWV_OK : ensure(ctx, ctx->degrid, padded + extra);
    if (rc) return rc;
    double2* G = (double2*)ctx->degrid.p;
    double* base = (double*)((char*)ctx->degrid.p + padded);
    double* sn = base + n_pix;
    double* hx = sn + n_pix;
    double* hy = hx + nx;
    k_hat_1d<<<(unsigned)((nx + ny + kDgBlock / 64 - 1) / (kDgBlock / 64)), kDgBlock, 0, s>>>(
        nx, ny, Nx, Ny, quad, hx);
    k_degrid_prep<<<blocks_of(n_pix), kDgBlock, 0, s>>>(nx, ny, cell, c, dw, image, hx, hy, quad,
                                                        base, sn);
    k_fill_planes<<<blocks_of(nq * cells), kDgBlock, 0, s>>>(nx, ny, Nx, Ny, nq, w0, dw, sign,
                                                             base, sn, G);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "swv_predict_degrid: plane fill");
    // batched 2-D transforms of the planes (plan cached per context and shape)
    if (!ctx->fft_plan || ctx->fft_shape[0] != Nx || ctx->fft_shape[1] != Ny) {
        destroy_fft_plan(ctx->fft_plan);
        ctx->fft_plan = nullptr;
        hipfftHandle plan = nullptr;
        int n2[2] = {Ny, Nx};
        if (hipfftPlanMany(&plan, 2, n2, nullptr, 1, (int)cells, nullptr, 1, (int)cells,
                           HIPFFT_Z2Z, (int)batch) != HIPFFT_SUCCESS)
            return fail(SWV_EHIP, "swv_predict_degrid: hipfftPlanMany failed");
        ctx->fft_plan = (void*)plan;
        ctx->fft_shape[0] = Nx;
        ctx->fft_shape[1] = Ny;
    }
    hipfftHandle plan = (hipfftHandle)ctx->fft_plan;
    bool ok = hipfftSetStream(plan, s) == HIPFFT_SUCCESS;
    for (int64_t q = 0; q < nq && ok; q += batch) {
        hipfftDoubleComplex* p = (hipfftDoubleComplex*)(G + q * cells);
        ok = hipfftExecZ2Z(plan, p, p, sign < 0 ? HIPFFT_FORWARD : HIPFFT_BACKWARD) == HIPFFT_SUCCESS;
    }
    if (!ok) return fail(SWV_EHIP, "swv_predict_degrid: hipfftExecZ2Z failed");
    kDegrid[support](s, n_vis, u, v, w, Nx, Ny, nq, cell, w0, dw, c, beta, sign, G,
                     (double2*)vis_out,
                     sort ? (char*)ctx->degrid.p + padded + extra : nullptr);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "swv_predict_degrid: degrid");
    if (stats) {
        stats->n_planes = nq;
        stats->grid_nx = Nx;
        stats->grid_ny = Ny;
        stats->w0 = w0;
        stats->dw = dw;
        stats->c = c;
        stats->plane_bytes = (int64_t)plane_bytes;
        stats->host_ms =
            std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0)
                .count();
    }
    clear_error();
    return SWV_OK;
}
