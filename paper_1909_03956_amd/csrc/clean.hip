// Clean loop (sections 2.1, 2.2, 3.5): image grids, dirty images and the
// dirty beam from the exact adjoint, the Hogbom minor cycle (Eqs. 4, 5), the
// clean image (Eq. 6) and the major-cycle driver around the tree predictor.
#include <hip/hip_cooperative_groups.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <climits>
#include <cmath>
#include <vector>

#include "api_internal.h"
#include "clean.h"
#include "sphere.h"
#include "tree.h"

namespace swv {

namespace {

constexpr int kGridBlock = 256;

// Direction of grid pixel p (SIN projection); off the unit disk: zeros.
__device__ __forceinline__ bool grid_direction(int64_t p, int nx, int cx, int cy, double cell,
                                               double& l, double& m, double& nm1) {
    const int64_t iy = p / nx, ix = p - iy * nx;
    l = (double)(ix - cx) * cell;
    m = (double)(iy - cy) * cell;
    const double r2 = l * l + m * m;
    const bool in = r2 < 1.0;
    nm1 = in ? -r2 / (1.0 + sqrt(1.0 - r2)) : 0.0;
    if (!in) l = m = 0.0;
    return in;
}

__global__ __launch_bounds__(kGridBlock) void k_grid(int64_t n, int nx, int cx, int cy,
                                                     double cell, double* __restrict__ l,
                                                     double* __restrict__ m,
                                                     double* __restrict__ nm1) {
    const int64_t p = (int64_t)blockIdx.x * kGridBlock + threadIdx.x;
    if (p >= n) return;
    double a, b, c;
    grid_direction(p, nx, cx, cy, cell, a, b, c);
    l[p] = a;
    m[p] = b;
    nm1[p] = c;
}

__global__ __launch_bounds__(kGridBlock) void k_fill_unit(int64_t n, double2* __restrict__ y) {
    const int64_t j = (int64_t)blockIdx.x * kGridBlock + threadIdx.x;
    if (j < n) y[j] = make_double2(1.0, 0.0);
}

// img[p] = Re x[p] / n_vis on the disk, 0 off it.
__global__ __launch_bounds__(kGridBlock) void k_real_image(int64_t n, const double2* __restrict__ x,
                                                           int nx, int cx, int cy, double cell,
                                                           double n_vis,
                                                           double* __restrict__ img) {
    const int64_t p = (int64_t)blockIdx.x * kGridBlock + threadIdx.x;
    if (p >= n) return;
    double l, m, nm1;
    const bool in = grid_direction(p, nx, cx, cy, cell, l, m, nm1);
    img[p] = in ? x[p].x / n_vis : 0.0;
}

// ---------------------------------------------------------------- Hogbom ---
// One workgroup runs the whole minor cycle.  Thread t owns pixels t, t + 1024,
// ... for the whole cycle, so a pixel is only ever read and written by its
// owner.  Each iteration: the owners' running peaks are reduced to the block's
// peak (largest key, lowest pixel id on ties: a total order, so the result
// does not depend on the reduction's shape), and one pass over the pixels
// subtracts the shifted beam and finds the next running peaks.  One barrier
// per iteration: the per-wave results alternate between two LDS slots.  Latency
// bound: 40 x 40 pixels 3.3 -> 2.3 us per iteration (DPP reductions).
constexpr int kHogBlock = 1024;
constexpr int kHogWaves = kHogBlock / 64;
constexpr int kHogBatch = 8;

__device__ __forceinline__ bool ahead(double k1, int i1, double k2, int i2) {
    return k1 > k2 || (k1 == k2 && i1 < i2);
}

// x of the lane that `CTRL` names (DPP, within rows of 16 lanes).
template <int CTRL>
__device__ __forceinline__ int dpp(int x) {
    return __builtin_amdgcn_mov_dpp(x, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp(double x) {
    return __hiloint2double(dpp<CTRL>(__double2hiint(x)), dpp<CTRL>(__double2loint(x)));
}
__device__ __forceinline__ int lane_value(int x, int lane) {
    return __builtin_amdgcn_readlane(x, lane);
}
__device__ __forceinline__ double lane_value(double x, int lane) {
    return __hiloint2double(lane_value(__double2hiint(x), lane),
                            lane_value(__double2loint(x), lane));
}

// op over groups of W lanes, W = 4, 16 or 64; the result is in every lane.
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppMirror = 0x140;
template <int W, class T, class Op>
__device__ __forceinline__ T over_lanes(T x, Op op) {
    x = op(x, dpp<kDppXor1>(x));
    x = op(x, dpp<kDppXor2>(x));
    if constexpr (W >= 16) {
        x = op(x, dpp<kDppHalfMirror>(x));
        x = op(x, dpp<kDppMirror>(x));
    }
    if constexpr (W == 64)
        x = op(op(lane_value(x, 0), lane_value(x, 16)), op(lane_value(x, 32), lane_value(x, 48)));
    return x;
}

// The best (key, val, idx) of W lanes, for all of them (W < 64: the groups hold
// the same): the largest key, then the lowest index that has it, then that lane's
// value, each by itself.  A third of the dependent steps of a butterfly of all three.
template <int W>
__device__ __forceinline__ void lanes_best(double& key, double& val, int& idx) {
    const double k = over_lanes<W>(key, [](double a, double b) { return a > b ? a : b; });
    const int i = over_lanes<W>(key == k ? idx : INT_MAX,
                                [](int a, int b) { return a < b ? a : b; });
    const unsigned long long who = __ballot(key == k && idx == i);
    const int lane = __builtin_amdgcn_readfirstlane(__ffsll(who) - 1);
    key = lane_value(key, lane);
    val = lane_value(val, lane);
    idx = i;
}

// The workgroup's best for every thread: waves, then their results by way of LDS.
// One barrier: a call may use the arrays again once another call lies between.
template <int WAVES>
__device__ __forceinline__ void block_best(double& key, double& val, int& idx, double* sk,
                                           double* sv, int* si) {
    lanes_best<64>(key, val, idx);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) {
        sk[wave] = key;
        sv[wave] = val;
        si[wave] = idx;
    }
    __syncthreads();
    key = sk[lane & (WAVES - 1)];
    val = sv[lane & (WAVES - 1)];
    idx = si[lane & (WAVES - 1)];
    lanes_best<WAVES>(key, val, idx);
}

template <bool ABS>
__global__ __launch_bounds__(kHogBlock) void k_hogbom(
    double* __restrict__ img, const double* __restrict__ beam, int nx, int ny, double gain,
    double threshold, int64_t max_iter, int64_t* __restrict__ comp_pix,
    double* __restrict__ comp_val, int64_t* __restrict__ n_found) {
    __shared__ double s_key[2][kHogWaves], s_val[2][kHogWaves];
    __shared__ int s_idx[2][kHogWaves];
    const int tid = threadIdx.x;
    const int n = nx * ny;
    const int64_t bw = 2 * (int64_t)nx - 1;
    // the thread's first pixel and the stride as (rows, columns)
    const int y0 = tid / nx, x0 = tid - (tid / nx) * nx;
    const int sy = kHogBlock / nx, sx = kHogBlock - sy * nx;

    double key = -HUGE_VAL, val = 0.0;
    int idx = INT_MAX;
    for (int p = tid; p < n; p += kHogBlock) {
        const double x = img[p];
        const double k = ABS ? fabs(x) : x;
        if (k > key) {
            key = k;
            val = x;
            idx = p;
        }
    }
    int64_t it = 0;
    for (int buf = 0;; buf ^= 1) {
        block_best<kHogWaves>(key, val, idx, s_key[buf], s_val[buf], s_idx[buf]);
        // the same decision in every thread
        if (it >= max_iter || !(key > threshold)) break;
        const double gc = gain * val;
        if (tid == 0) {
            comp_pix[it] = idx;
            comp_val[it] = gc;
        }
        ++it;
        const int py = idx / nx, px = idx - (idx / nx) * nx;
        const double* B = beam + (int64_t)(ny - 1 - py) * bw + (nx - 1 - px);
        key = -HUGE_VAL;
        val = 0.0;
        idx = INT_MAX;
        int y = y0, x = x0;
        // kHogBatch pixels per step: their loads are all in flight together
        for (int p0 = tid; p0 < n; p0 += kHogBatch * kHogBlock) {
            double iv[kHogBatch], bv[kHogBatch];
#pragma unroll
            for (int b = 0; b < kHogBatch; ++b) {
                const int p = p0 + b * kHogBlock;
                if (p < n) {
                    iv[b] = img[p];
                    bv[b] = B[(int64_t)y * bw + x];
                }
                x += sx;
                y += sy;
                if (x >= nx) {
                    x -= nx;
                    ++y;
                }
            }
#pragma unroll
            for (int b = 0; b < kHogBatch; ++b) {
                const int p = p0 + b * kHogBlock;
                if (p < n) {
                    const double t = gc * bv[b];
                    const double r = iv[b] - t;
                    img[p] = r;
                    const double k = ABS ? fabs(r) : r;
                    if (k > key) {
                        key = k;
                        val = r;
                        idx = p;
                    }
                }
            }
        }
    }
    if (tid == 0) *n_found = it;
}

// The same minor cycle spread over G workgroups, all resident at once (a
// cooperative launch: the runtime refuses a grid that could not be).  Global
// thread g owns pixels g, g + G B, ...  Each iteration a workgroup publishes
// its peak in its slot and gathers every workgroup's slot of that iteration:
// the gather is the barrier, with no shared counter.  Every workgroup reduces
// the G peaks in the same total order, so all take the same decision.  Slots
// alternate between two buffers: a workgroup can only reuse a buffer after every
// other one has published the next iteration, i.e. finished reading it.  Every
// wait is bounded: after kHogSpinLimit polls the workgroup gives up, the cycle
// ends and *n_found is set to -1.
//
// A slot is three 64-bit words, each with 32 bits of the peak (value high, value
// low, index) beside the iteration's low 32 bits: a word with the right number is
// of that iteration whatever the others are, so the words need no order among
// themselves, and nothing else passes between workgroups (a pixel belongs to one
// thread).  Ordered by release and acquire instead, each exchange would write
// back and drop the caches that hold image and beam.  Bound by the exchange's and
// the loads' latency: 256 x 256 pixels 5.45 -> 4.12 us per iteration, 1024 x 1024
// 26 -> 11.1.
constexpr int kHogGridBlock = 256;
constexpr int kHogGridWaves = kHogGridBlock / 64;
constexpr int kHogGridBatch = 2;
constexpr int kHogSpinLimit = 1 << 23;

// slot layout: [buffer][workgroup][value high, value low, index, unused], the
// iteration's number + 1 in the upper half of each 64-bit word
__device__ __forceinline__ void publish(unsigned long long* slot, double val, int idx,
                                        unsigned tag) {
    const unsigned long long t = (unsigned long long)tag << 32;
    const unsigned long long x = (unsigned long long)__double_as_longlong(val);
    __hip_atomic_store(slot + 0, t | (x >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(slot + 1, t | (x & 0xffffffffull), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(slot + 2, t | (unsigned)idx, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits for the slot's words of iteration `tag`; false if they do not come.
__device__ __forceinline__ bool await(const unsigned long long* slot, unsigned tag, double& val,
                                      int& idx) {
    for (int spins = 0; spins <= kHogSpinLimit; ++spins) {
        unsigned long long a[3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
            a[i] = __hip_atomic_load(slot + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((unsigned)(a[0] >> 32) == tag && (unsigned)(a[1] >> 32) == tag &&
            (unsigned)(a[2] >> 32) == tag) {
            val = __longlong_as_double((long long)(a[0] << 32 | (a[1] & 0xffffffffull)));
            idx = (int)(unsigned)a[2];
            return true;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return false;
}

template <bool ABS>
__global__ __launch_bounds__(kHogGridBlock) void k_hogbom_grid(
    double* __restrict__ img, const double* __restrict__ beam, int nx, int ny, double gain,
    double threshold, int64_t max_iter, int64_t* __restrict__ comp_pix,
    double* __restrict__ comp_val, int64_t* __restrict__ n_found,
    unsigned long long* __restrict__ slots) {
    __shared__ double sk[2][kHogGridWaves], sv[2][kHogGridWaves];
    __shared__ int si[2][kHogGridWaves];
    __shared__ int s_timeout;
    const int G = (int)gridDim.x;
    const int n = nx * ny;
    const int64_t bw = 2 * (int64_t)nx - 1;
    const int stride = G * kHogGridBlock;
    const int g0 = (int)blockIdx.x * kHogGridBlock + (int)threadIdx.x;
    const int y0 = g0 / nx, x0 = g0 - (g0 / nx) * nx;
    const int sy = stride / nx, sx = stride - sy * nx;
    if (threadIdx.x == 0) s_timeout = 0;

    double key = -HUGE_VAL, val = 0.0;
    int idx = INT_MAX;
    for (int p = g0; p < n; p += stride) {
        const double x = img[p];
        const double k = ABS ? fabs(x) : x;
        if (k > key) {
            key = k;
            val = x;
            idx = p;
        }
    }
    int64_t it = 0;   // the peaks being exchanged belong to the image after `it` components
    for (;;) {
        block_best<kHogGridWaves>(key, val, idx, sk[0], sv[0], si[0]);
        unsigned long long* buf = slots + (size_t)(it & 1) * 4 * G;
        const unsigned tag = (unsigned)(it + 1);
        if (threadIdx.x == 0) publish(buf + 4 * (size_t)blockIdx.x, val, idx, tag);
        // gather: thread b waits for workgroup b's slot of this iteration
        key = -HUGE_VAL;
        val = 0.0;
        idx = INT_MAX;
        for (int b = threadIdx.x; b < G; b += kHogGridBlock) {
            double v2;
            int i2;
            if (!await(buf + 4 * (size_t)b, tag, v2, i2)) {
                s_timeout = 1;
                continue;
            }
            const double k2 = i2 == INT_MAX ? -HUGE_VAL : (ABS ? fabs(v2) : v2);
            if (ahead(k2, i2, key, idx)) {
                key = k2;
                val = v2;
                idx = i2;
            }
        }
        // its barrier also publishes s_timeout
        block_best<kHogGridWaves>(key, val, idx, sk[1], sv[1], si[1]);
        if (s_timeout) {
            if (threadIdx.x == 0) *n_found = -1;
            return;
        }
        if (it >= max_iter || !(key > threshold)) break;   // the same in every workgroup
        const double gc = gain * val;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            comp_pix[it] = idx;
            comp_val[it] = gc;
        }
        ++it;
        const int py = idx / nx, px = idx - (idx / nx) * nx;
        const double* B = beam + (int64_t)(ny - 1 - py) * bw + (nx - 1 - px);
        key = -HUGE_VAL;
        val = 0.0;
        idx = INT_MAX;
        int y = y0, x = x0;
        // kHogGridBatch pixels per step: their loads are all in flight together
        for (int p0 = g0; p0 < n; p0 += kHogGridBatch * stride) {
            double iv[kHogGridBatch], bv[kHogGridBatch];
#pragma unroll
            for (int b = 0; b < kHogGridBatch; ++b) {
                if (b * stride < n - p0) {
                    iv[b] = img[p0 + b * stride];
                    bv[b] = B[(int64_t)y * bw + x];
                }
                x += sx;
                y += sy;
                if (x >= nx) {
                    x -= nx;
                    ++y;
                }
            }
#pragma unroll
            for (int b = 0; b < kHogGridBatch; ++b)
                if (b * stride < n - p0) {
                    const int p = p0 + b * stride;
                    const double t = gc * bv[b];
                    const double r = iv[b] - t;
                    img[p] = r;
                    const double k = ABS ? fabs(r) : r;
                    if (k > key) {
                        key = k;
                        val = r;
                        idx = p;
                    }
                }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *n_found = it;
}

// --------------------------------------------------------------- restore ---
// Components are staged through LDS in tiles (pixel split into row and
// column once per component); each thread sums its pixel's terms in list
// order.
constexpr int kRestTile = 256;

__global__ __launch_bounds__(kGridBlock) void k_restore(
    int nx, int64_t n, int64_t n_comp, const int64_t* __restrict__ comp_pix,
    const double* __restrict__ comp_val, double a, double b, double c,
    const double* __restrict__ residual, double* __restrict__ out) {
    __shared__ double s_x[kRestTile], s_y[kRestTile], s_g[kRestTile];
    const int64_t p = (int64_t)blockIdx.x * kGridBlock + threadIdx.x;
    const int64_t pc = p < n ? p : n - 1;
    const double iy = (double)(pc / nx), ix = (double)(pc - (pc / nx) * nx);
    const double b2 = 2.0 * b;
    double s = 0.0;
    for (int64_t t0 = 0; t0 < n_comp; t0 += kRestTile) {
        const int nt = (int)(n_comp - t0 < kRestTile ? n_comp - t0 : kRestTile);
        __syncthreads();
        for (int i = threadIdx.x; i < nt; i += kGridBlock) {
            const int64_t q = comp_pix[t0 + i];
            s_y[i] = (double)(q / nx);
            s_x[i] = (double)(q - (q / nx) * nx);
            s_g[i] = comp_val[t0 + i];
        }
        __syncthreads();
        for (int i = 0; i < nt; ++i) {
            const double dx = ix - s_x[i], dy = iy - s_y[i];
            s += s_g[i] * exp(-(a * dx * dx + b2 * dx * dy + c * dy * dy));
        }
    }
    if (p < n) out[p] = residual ? s + residual[p] : s;
}

unsigned grid_blocks(int64_t n) { return (unsigned)((n + kGridBlock - 1) / kGridBlock); }

__global__ void k_zero_u64(int64_t n, unsigned long long* p) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

// From how many pixels the cycle runs grid-wide: one workgroup takes 2.6, 3.2 and
// 4.7 us per iteration at 64^2, 80^2 and 100^2 pixels, the grid 2.8, 2.9 and 3.2.
// A capture records one workgroup up to 16,383 pixels: a cooperative launch may not
// be capturable.
constexpr int kHogGridMinPixels = 5120, kHogGridMinCaptured = 16384;
// Two pixels per thread (one: 4.7 us at 256^2 against 4.1, four: 3.8 at 160^2
// against 3.5) and up to 256 workgroups of 256 (64 and 128 take 31 and 17 us at
// 1024^2 against 11); each waits for every other, one slot per thread.
constexpr int kHogGridPerThread = 2, kHogGridMaxBlocks = 256;

bool coop_supported(int device) {
    int v = 0;
    return hipDeviceGetAttribute(&v, hipDeviceAttributeCooperativeLaunch, device) == hipSuccess &&
           v != 0;
}

bool hogbom_grid_wide(swv_ctx ctx, int n, int flags) {
    if (n < kHogGridMinPixels || (flags & SWV_HOGBOM_SINGLE) || !coop_supported(ctx->device))
        return false;
    return n >= kHogGridMinCaptured || !stream_captured(ctx);
}

int check_grid(int nx, int ny, double cell) {
    if (nx < 1 || ny < 1 || nx > 32768 || ny > 32768 || (int64_t)nx * ny > (1 << 30))
        return fail(SWV_EINVAL, "grid %d x %d outside 1 .. 32768 per side, 2^30 pixels", nx, ny);
    if (!(cell > 0.0) || !std::isfinite(cell))
        return fail(SWV_EDOMAIN, "grid cell must be positive and finite");
    return SWV_OK;
}

// Rows go through in slabs whose tables stay within kGridSlabBytes (at least one
// row): 256 MB, what the last-level cache holds, and rows enough for the
// workgroups to run for long (a 256 x 256 image: 62,000).
constexpr size_t kGridSlabBytes = size_t(256) << 20;

// The FP64 dirty image by axis phasors.
int grid_image(swv_ctx ctx, const GridGeom& g, const GridPlan& p, int64_t n_vis, const double* u,
               const double* v, const double* w, const void* y, int nx, int ny, int cx, int cy,
               int sign, double* img) {
    const int64_t cap = std::max<int64_t>(1, (int64_t)(kGridSlabBytes / grid_row_bytes(g)));
    const int64_t n_slabs = (n_vis + cap - 1) / cap;
    const int64_t rows = (n_vis + n_slabs - 1) / n_slabs;
    const int64_t chunk = grid_chunk(g, p, rows, ctx->n_cu);
    const int64_t n_chunks = (rows + chunk - 1) / chunk;
    int rc = ensure(ctx, ctx->grid, grid_slab_bytes(g, rows));
    if (!rc) rc = ensure(ctx, ctx->partial, grid_partial_bytes(g, n_chunks));
    if (rc) return rc;
    double* part = (double*)ctx->partial.p;
    for (int64_t j = 0; j < n_vis; j += rows) {
        const int64_t nr = std::min<int64_t>(rows, n_vis - j);
        const hipError_t e =
            launch_grid_slab(ctx->stream, g, p, nr, chunk, u + j, v + j, w + j,
                             y ? (const double2*)y + j : nullptr, sign, j > 0, ctx->grid.p, part);
        if (e != hipSuccess) return hip_fail(e, "swv_dirty_image");
    }
    const hipError_t e = launch_grid_finish(ctx->stream, g, SWV_FP64, part, n_chunks, nx, ny, cx, cy, n_vis, img);
    return e == hipSuccess ? SWV_OK : hip_fail(e, "swv_dirty_image");
}

}  // namespace

}  // namespace swv

using namespace swv;

#define CLEAN_CHECK_CTX(ctx) \
    if (!(ctx)) return fail(SWV_EINVAL, "%s: null context", __func__)
#define CLEAN_GUARD(ctx)                   \
    DeviceGuard guard_((ctx)->device);     \
    if (!guard_.ok) return fail(SWV_EHIP, "%s: cannot select device %d", __func__, (ctx)->device)
#define CLEAN_HIP(expr)                                      \
    do {                                                     \
        hipError_t e_ = (expr);                              \
        if (e_ != hipSuccess) return hip_fail(e_, #expr);    \
    } while (0)
#define CLEAN_RC(expr)          \
    do {                        \
        const int rc_ = (expr); \
        if (rc_) return rc_;    \
    } while (0)

extern "C" int swv_image_grid(swv_ctx ctx, int nx, int ny, int cx, int cy, double cell,
                              double* l, double* m, double* nm1) {
    CLEAN_CHECK_CTX(ctx);
    CLEAN_RC(check_grid(nx, ny, cell));
    if (!l || !m || !nm1) return fail(SWV_EINVAL, "swv_image_grid: null output");
    CLEAN_GUARD(ctx);
    const int64_t n = (int64_t)nx * ny;
    k_grid<<<grid_blocks(n), kGridBlock, 0, ctx->stream>>>(n, nx, cx, cy, cell, l, m, nm1);
    CLEAN_HIP(hipGetLastError());
    return SWV_OK;
}

extern "C" int swv_dirty_image(swv_ctx ctx, int64_t n_vis, const double* u, const double* v,
                               const double* w, const void* y, int nx, int ny, int cx, int cy,
                               double cell, int sign, int prec, double* img_out) {
    CLEAN_CHECK_CTX(ctx);
    CLEAN_RC(check_grid(nx, ny, cell));
    if (n_vis < 1) return fail(SWV_EINVAL, "swv_dirty_image: no visibilities");
    if (!u || !v || !w || !img_out) return fail(SWV_EINVAL, "swv_dirty_image: null argument");
    if (sign != 1 && sign != -1) return fail(SWV_EDOMAIN, "sign must be +1 or -1 (got %d)", sign);
    if (prec != SWV_FP64 && prec != SWV_F32C)
        return fail(SWV_EINVAL, "swv_dirty_image: unsupported precision %d", prec);
    CLEAN_GUARD(ctx);
    GridGeom geom;
    GridPlan plan;
    if (grid_plan(nx, ny, cx, cy, cell, prec, &geom, &plan)) {
        if (prec == SWV_FP64)
            return grid_image(ctx, geom, plan, n_vis, u, v, w, y, nx, ny, cx, cy, sign, img_out);
        // in the adjoint's chunks of rows, whose Kahan sums these are
        const AdjointShape sh = adjoint_shape(ctx, n_vis, (int64_t)nx * ny, prec);
        CLEAN_RC(ensure(ctx, ctx->partial, grid_partial_bytes(geom, sh.n_chunks)));
        double* part = (double*)ctx->partial.p;
        CLEAN_HIP(launch_image_f32c(ctx->stream, geom, plan, n_vis, sh.chunk, ctx->n_cu, u, v, w, y, sign,
                                    part));
        CLEAN_HIP(launch_grid_finish(ctx->stream, geom, prec, part, sh.n_chunks, nx, ny, cx, cy, n_vis,
                                     img_out));
        return SWV_OK;
    }
    const int64_t n = (int64_t)nx * ny;
    CLEAN_RC(ensure(ctx, ctx->grid, 40 * (size_t)n));
    // the complex adjoint output first, so that it is 16-byte aligned for any n
    double2* gx = (double2*)ctx->grid.p;
    double* gl = (double*)(gx + n);
    double* gm = gl + n;
    double* gn = gm + n;
    const double2* yy = (const double2*)y;
    if (!yy) {
        if (ctx->ones.n < 16 * (size_t)n_vis) {
            CLEAN_RC(ensure(ctx, ctx->ones, 16 * (size_t)n_vis));
            // fill the whole buffer: later calls with fewer rows reuse it
            const int64_t cap = (int64_t)(ctx->ones.n / 16);
            k_fill_unit<<<grid_blocks(cap), kGridBlock, 0, ctx->stream>>>(cap, (double2*)ctx->ones.p);
            CLEAN_HIP(hipGetLastError());
        }
        yy = (const double2*)ctx->ones.p;
    }
    k_grid<<<grid_blocks(n), kGridBlock, 0, ctx->stream>>>(n, nx, cx, cy, cell, gl, gm, gn);
    CLEAN_HIP(hipGetLastError());
    CLEAN_RC(swv_adjoint(ctx, n_vis, u, v, w, yy, n, gl, gm, gn, sign, prec, gx));
    k_real_image<<<grid_blocks(n), kGridBlock, 0, ctx->stream>>>(n, gx, nx, cx, cy, cell,
                                                                 (double)n_vis, img_out);
    CLEAN_HIP(hipGetLastError());
    return SWV_OK;
}

extern "C" int swv_hogbom(swv_ctx ctx, int nx, int ny, double* image, const double* beam,
                          double gain, double threshold, int64_t max_iter, int flags,
                          int64_t* comp_pix, double* comp_val, int64_t* n_found) {
    CLEAN_CHECK_CTX(ctx);
    CLEAN_RC(check_grid(nx, ny, 1.0));
    if (!image || !beam || !n_found) return fail(SWV_EINVAL, "swv_hogbom: null argument");
    if (max_iter < 0) return fail(SWV_EINVAL, "swv_hogbom: negative max_iter");
    if (max_iter > 0 && (!comp_pix || !comp_val))
        return fail(SWV_EINVAL, "swv_hogbom: null component arrays");
    if (!std::isfinite(gain) || std::isnan(threshold))
        return fail(SWV_EDOMAIN, "swv_hogbom: gain must be finite, threshold a number");
    if (flags & ~(SWV_HOGBOM_ABS | SWV_HOGBOM_SINGLE))
        return fail(SWV_EINVAL, "swv_hogbom: unknown flags %d", flags);
    CLEAN_GUARD(ctx);
    const int n = nx * ny;
    if (hogbom_grid_wide(ctx, n, flags)) {
        constexpr int per = kHogGridPerThread * kHogGridBlock;
        int G = (n + per - 1) / per;
        G = G < kHogGridMaxBlocks ? G : kHogGridMaxBlocks;
        G = G < ctx->n_cu ? G : ctx->n_cu;
        CLEAN_RC(ensure(ctx, ctx->hog, 64 * (size_t)G));
        unsigned long long* slots = (unsigned long long*)ctx->hog.p;
        // iteration numbers start from a clean slate (a fill kernel, no memset)
        k_zero_u64<<<(unsigned)((8 * G + 255) / 256), 256, 0, ctx->stream>>>(8 * (int64_t)G, slots);
        CLEAN_HIP(hipGetLastError());
        void* args[] = {&image, (void*)&beam, &nx, &ny, &gain, &threshold, &max_iter, &comp_pix,
                        &comp_val, &n_found, &slots};
        const void* fn = (flags & SWV_HOGBOM_ABS) ? (const void*)k_hogbom_grid<true>
                                                  : (const void*)k_hogbom_grid<false>;
        const hipError_t e = hipLaunchCooperativeKernel(fn, dim3(G), dim3(kHogGridBlock), args, 0,
                                                        ctx->stream);
        if (e == hipSuccess) return SWV_OK;
        // a grid that cannot be resident at once is refused before it starts
        (void)hipGetLastError();
    }
    if (flags & SWV_HOGBOM_ABS)
        k_hogbom<true><<<1, kHogBlock, 0, ctx->stream>>>(image, beam, nx, ny, gain, threshold,
                                                         max_iter, comp_pix, comp_val, n_found);
    else
        k_hogbom<false><<<1, kHogBlock, 0, ctx->stream>>>(image, beam, nx, ny, gain, threshold,
                                                          max_iter, comp_pix, comp_val, n_found);
    CLEAN_HIP(hipGetLastError());
    return SWV_OK;
}

extern "C" int swv_cross_reference(int J, double ra_p, double dec_p, int nx, int ny, double cell,
                                   int64_t* pix) {
    if (J < 1 || J > SWV_MAX_LEVEL) return fail(SWV_EDOMAIN, "J = %d outside [1, 29]", J);
    CLEAN_RC(check_grid(nx, ny, cell));
    if (!pix) return fail(SWV_EINVAL, "swv_cross_reference: null pix");
    if (!std::isfinite(ra_p) || !std::isfinite(dec_p))
        return fail(SWV_EDOMAIN, "swv_cross_reference: non-finite phase centre");
    CLEAN_RC(cross_reference(J, ra_p, dec_p, nx, ny, cell, pix));
    clear_error();
    return SWV_OK;
}

extern "C" int swv_tree_build_pixels(int J, double ra_p, double dec_p, int64_t n,
                                     const int64_t* pix, const double* flux, swv_tree* out) {
    if (!out) return fail(SWV_EINVAL, "swv_tree_build_pixels: null out");
    *out = nullptr;
    if (J < 1 || J > SWV_MAX_LEVEL) return fail(SWV_EDOMAIN, "J = %d outside [1, 29]", J);
    if (n < 0) return fail(SWV_EINVAL, "swv_tree_build_pixels: negative n");
    if (n > 0 && (!pix || !flux)) return fail(SWV_EINVAL, "swv_tree_build_pixels: null array");
    if (!std::isfinite(ra_p) || !std::isfinite(dec_p))
        return fail(SWV_EDOMAIN, "swv_tree_build_pixels: non-finite phase centre");
    const int64_t np = n_pixels(J);
    for (int64_t i = 0; i < n; ++i) {
        if (pix[i] < 0 || pix[i] >= np)
            return fail(SWV_EDOMAIN, "swv_tree_build_pixels: pixel %lld outside level %d",
                        (long long)pix[i], J);
        if (!std::isfinite(flux[i]))
            return fail(SWV_EDOMAIN, "swv_tree_build_pixels: non-finite flux at %lld",
                        (long long)i);
    }
    try {
        auto* t = new swv_tree_s();
        const int rc = build_tree_pixels(J, ra_p, dec_p, n, pix, flux, t);
        if (rc) {
            delete t;
            return rc;
        }
        *out = t;
    } catch (const std::bad_alloc&) {
        return fail(SWV_ENOMEM, "swv_tree_build_pixels: host allocation failed");
    }
    clear_error();
    return SWV_OK;
}

extern "C" int swv_fit_clean_beam(int nbx, int nby, const double* beam, double* abc) {
    if (nbx < 1 || nby < 1 || !beam || !abc) return fail(SWV_EINVAL, "swv_fit_clean_beam: bad argument");
    for (int64_t i = 0; i < (int64_t)nbx * nby; ++i)
        if (!std::isfinite(beam[i])) return fail(SWV_EDOMAIN, "swv_fit_clean_beam: non-finite beam");
    try {
        CLEAN_RC(fit_clean_beam(nbx, nby, beam, abc));
    } catch (const std::bad_alloc&) {
        return fail(SWV_ENOMEM, "swv_fit_clean_beam: host allocation failed");
    }
    clear_error();
    return SWV_OK;
}

extern "C" int swv_restore(swv_ctx ctx, int nx, int ny, int64_t n_comp, const int64_t* comp_pix,
                           const double* comp_val, const double* abc, const double* residual,
                           double* out) {
    CLEAN_CHECK_CTX(ctx);
    CLEAN_RC(check_grid(nx, ny, 1.0));
    if (n_comp < 0) return fail(SWV_EINVAL, "swv_restore: negative n_comp");
    if (!abc || !out || (n_comp > 0 && (!comp_pix || !comp_val)))
        return fail(SWV_EINVAL, "swv_restore: null argument");
    if (!std::isfinite(abc[0]) || !std::isfinite(abc[1]) || !std::isfinite(abc[2]))
        return fail(SWV_EDOMAIN, "swv_restore: non-finite beam parameters");
    CLEAN_GUARD(ctx);
    const int64_t n = (int64_t)nx * ny;
    k_restore<<<grid_blocks(n), kGridBlock, 0, ctx->stream>>>(nx, n, n_comp, comp_pix, comp_val,
                                                              abc[0], abc[1], abc[2], residual, out);
    CLEAN_HIP(hipGetLastError());
    return SWV_OK;
}

namespace {

// Owns the per-call device scratch and events of swv_wavelet_clean.
struct CleanScratch {
    void* p[5] = {};
    hipEvent_t ev[2] = {};
    swv_tree tree = nullptr;
    ~CleanScratch() {
        for (void* q : p)
            if (q) (void)hipFree(q);
        for (hipEvent_t e : ev)
            if (e) (void)hipEventDestroy(e);
        if (tree) (void)swv_tree_destroy(tree);
    }
};

}  // namespace

extern "C" int swv_wavelet_clean(swv_ctx ctx, const swv_clean_params_t* P, int64_t n_vis,
                                 const double* u, const double* v, const double* w,
                                 const void* vis_obs, double* beam, double* residual,
                                 void* vis_model, int64_t cap, int64_t* comp_pix,
                                 double* comp_val, int64_t* n_comp, swv_clean_stats_t* stats) {
    CLEAN_CHECK_CTX(ctx);
    if (!P) return fail(SWV_EINVAL, "swv_wavelet_clean: null params");
    CLEAN_RC(check_grid(P->nx, P->ny, P->cell));
    if (P->J < 1 || P->J > SWV_MAX_LEVEL) return fail(SWV_EDOMAIN, "J = %d outside [1, 29]", P->J);
    if (n_vis < 1 || !u || !v || !w || !vis_obs || !beam || !residual || !vis_model || !n_comp)
        return fail(SWV_EINVAL, "swv_wavelet_clean: null argument or no visibilities");
    if (P->minor_iter < 0 || P->n_major < 0 || P->n_major > SWV_CLEAN_MAX_CYCLES)
        return fail(SWV_EINVAL, "swv_wavelet_clean: minor_iter >= 0, 0 <= n_major <= %d",
                    SWV_CLEAN_MAX_CYCLES);
    const int64_t need = P->minor_iter * (int64_t)P->n_major;
    if (cap < need || (need > 0 && (!comp_pix || !comp_val)))
        return fail(SWV_EINVAL, "swv_wavelet_clean: component arrays hold %lld, need %lld",
                    (long long)cap, (long long)need);
    if (P->sign != 1 && P->sign != -1) return fail(SWV_EDOMAIN, "sign must be +1 or -1");
    if (P->predictor != SWV_PREDICT_TREE && P->predictor != SWV_PREDICT_DEGRID &&
        P->predictor != SWV_PREDICT_DIRECT)
        return fail(SWV_EINVAL, "swv_wavelet_clean: unknown predictor %d", P->predictor);
    if (P->image_prec != SWV_FP64 && P->image_prec != SWV_F32C)
        return fail(SWV_EINVAL, "swv_wavelet_clean: unsupported image precision %d",
                    P->image_prec);
    if (P->predictor == SWV_PREDICT_DEGRID && (P->support < 2 || P->support > 16))
        return fail(SWV_EINVAL, "swv_wavelet_clean: support %d outside 2 .. 16", P->support);
    if (!std::isfinite(P->gain) || std::isnan(P->threshold))
        return fail(SWV_EDOMAIN, "swv_wavelet_clean: gain must be finite, threshold a number");
    const int nx = P->nx, ny = P->ny;
    const int64_t n_pix = (int64_t)nx * ny;
    *n_comp = 0;
    if (stats) *stats = swv_clean_stats_t{};
    try {
        // components are cross-referenced to sphere pixels (section 3.5) as the
        // minor cycles find them: the table of every image pixel took 27 ms of
        // long-double arithmetic for 256 x 256, a thousand components 0.4 ms
        CLEAN_RC(check_on_disk(nx, ny, P->cell));
        CLEAN_GUARD(ctx);
        const hipStream_t s = ctx->stream;
        CleanScratch S;
        const int64_t ncap = need > 0 ? need : 1;
        CLEAN_HIP(hipMalloc(&S.p[0], 8 * (size_t)ncap));   // component pixels
        CLEAN_HIP(hipMalloc(&S.p[1], 8 * (size_t)ncap));   // component values
        CLEAN_HIP(hipMalloc(&S.p[2], 16 * (size_t)n_vis));  // residual visibilities
        CLEAN_HIP(hipMalloc(&S.p[3], 256));                 // n_found, chi^2
        CLEAN_HIP(hipEventCreate(&S.ev[0]));
        CLEAN_HIP(hipEventCreate(&S.ev[1]));
        int64_t* d_pix = (int64_t*)S.p[0];
        double* d_val = (double*)S.p[1];
        int64_t* d_found = (int64_t*)S.p[3];
        double* d_chi2 = (double*)S.p[3] + 1;
        const auto lap = [&](double* ms) -> int {
            CLEAN_HIP(hipEventRecord(S.ev[1], s));
            CLEAN_HIP(hipEventSynchronize(S.ev[1]));
            float t = 0.f;
            CLEAN_HIP(hipEventElapsedTime(&t, S.ev[0], S.ev[1]));
            if (ms) *ms = t;
            CLEAN_HIP(hipEventRecord(S.ev[0], s));
            return SWV_OK;
        };
        double scratch_ms = 0.0;
        CLEAN_HIP(hipEventRecord(S.ev[0], s));
        // the beam once, in the images' precision
        CLEAN_RC(swv_dirty_image(ctx, n_vis, u, v, w, nullptr, 2 * nx - 1, 2 * ny - 1, nx - 1,
                                 ny - 1, P->cell, P->sign, P->image_prec, beam));
        CLEAN_RC(lap(stats ? &stats->ms_beam : &scratch_ms));
        CLEAN_RC(swv_dirty_image(ctx, n_vis, u, v, w, vis_obs, nx, ny, nx / 2, ny / 2, P->cell,
                                 P->sign, P->image_prec, residual));
        CLEAN_RC(lap(stats ? &stats->ms_dirty : &scratch_ms));
        CLEAN_HIP(hipMemsetAsync(vis_model, 0, 16 * (size_t)n_vis, s));
        int64_t total = 0;
        std::vector<int64_t> kj;
        std::vector<double> model, ml, mm, mf;
        double* d_model = nullptr;
        if (P->predictor != SWV_PREDICT_TREE) {
            model.assign((size_t)n_pix, 0.0);
            CLEAN_HIP(hipMalloc(&S.p[4], 24 * (size_t)n_pix));
            d_model = (double*)S.p[4];
        }
        for (int cyc = 0; cyc < P->n_major; ++cyc) {
            CLEAN_RC(swv_hogbom(ctx, nx, ny, residual, beam, P->gain, P->threshold, P->minor_iter,
                                P->flags, d_pix + total, d_val + total, d_found));
            int64_t found = 0;
            CLEAN_HIP(hipMemcpyAsync(&found, d_found, 8, hipMemcpyDeviceToHost, s));
            double ms_minor = 0.0;
            CLEAN_RC(lap(&ms_minor));   // synchronises: `found` is valid
            if (found < 0)
                return fail(SWV_EHIP, "swv_wavelet_clean: the grid-wide minor cycle timed out");
            if (found == 0) break;
            CLEAN_HIP(hipMemcpyAsync(comp_pix + total, d_pix + total, 8 * (size_t)found,
                                     hipMemcpyDeviceToHost, s));
            CLEAN_HIP(hipMemcpyAsync(comp_val + total, d_val + total, 8 * (size_t)found,
                                     hipMemcpyDeviceToHost, s));
            CLEAN_HIP(hipStreamSynchronize(s));
            total += found;
            const auto t0 = std::chrono::steady_clock::now();
            int64_t leaves = 0;
            if (P->predictor == SWV_PREDICT_TREE) {
                // the model tree of every component so far, from the cross-referenced pixels
                const int64_t known = (int64_t)kj.size();
                kj.resize((size_t)total);
                cross_reference_pixels(P->J, P->ra_p, P->dec_p, nx, ny, P->cell, total - known,
                                       comp_pix + known, kj.data() + known);
                if (S.tree) {
                    (void)swv_tree_destroy(S.tree);   // the stream is idle here
                    S.tree = nullptr;
                }
                CLEAN_RC(swv_tree_build_pixels(P->J, P->ra_p, P->dec_p, total, kj.data(),
                                               comp_val, &S.tree));
                swv_tree_stats_t ts;
                (void)swv_tree_stats(S.tree, &ts);
                leaves = ts.n_leaves;
            } else {
                // the model image: components summed per pixel in list order
                std::fill(model.begin(), model.end(), 0.0);
                for (int64_t i = 0; i < total; ++i) model[(size_t)comp_pix[i]] += comp_val[i];
                if (P->predictor == SWV_PREDICT_DIRECT) {
                    ml.clear();
                    mm.clear();
                    mf.clear();
                    for (int64_t p = 0; p < n_pix; ++p)
                        if (model[(size_t)p] != 0.0) {
                            const int64_t iy = p / nx, ix = p - iy * nx;
                            ml.push_back((double)(ix - nx / 2) * P->cell);
                            mm.push_back((double)(iy - ny / 2) * P->cell);
                            mf.push_back(model[(size_t)p]);
                        }
                    leaves = (int64_t)mf.size();
                    for (const auto* a : {&ml, &mm, &mf}) {
                        const size_t k = (a == &ml ? 0 : a == &mm ? 1 : 2);
                        CLEAN_HIP(hipMemcpyAsync(d_model + k * (size_t)n_pix, a->data(),
                                                 8 * a->size(), hipMemcpyHostToDevice, s));
                    }
                } else {
                    for (int64_t p = 0; p < n_pix; ++p) leaves += model[(size_t)p] != 0.0;
                    CLEAN_HIP(hipMemcpyAsync(d_model, model.data(), 8 * (size_t)n_pix,
                                             hipMemcpyHostToDevice, s));
                }
            }
            const double ms_build =
                std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0)
                    .count();
            CLEAN_HIP(hipEventRecord(S.ev[0], s));
            if (P->predictor == SWV_PREDICT_TREE)
                CLEAN_RC(swv_predict_tree(ctx, S.tree, n_vis, u, v, w, P->sign, SWV_FP64,
                                          vis_model));
            else if (P->predictor == SWV_PREDICT_DEGRID)
                CLEAN_RC(swv_predict_degrid(ctx, nx, ny, P->cell, d_model, n_vis, u, v, w,
                                            P->support, P->sign, vis_model, nullptr));
            else
                CLEAN_RC(swv_predict_direct(ctx, n_vis, u, v, w, leaves, d_model,
                                            d_model + n_pix, d_model + 2 * n_pix, P->sign,
                                            SWV_FP64, vis_model));
            double ms_predict = 0.0, ms_image = 0.0;
            CLEAN_RC(lap(&ms_predict));
            CLEAN_RC(swv_residual_chi2(ctx, n_vis, vis_obs, vis_model, 1.0, S.p[2], d_chi2));
            CLEAN_RC(swv_dirty_image(ctx, n_vis, u, v, w, S.p[2], nx, ny, nx / 2, ny / 2,
                                     P->cell, P->sign, P->image_prec, residual));
            double chi2 = 0.0;
            CLEAN_HIP(hipMemcpyAsync(&chi2, d_chi2, 8, hipMemcpyDeviceToHost, s));
            CLEAN_RC(lap(&ms_image));
            if (stats) {
                stats->found[cyc] = found;
                stats->leaves[cyc] = leaves;
                stats->chi2[cyc] = chi2;
                stats->ms_minor[cyc] = ms_minor;
                stats->ms_build[cyc] = ms_build;
                stats->ms_predict[cyc] = ms_predict;
                stats->ms_image[cyc] = ms_image;
                stats->n_cycles = cyc + 1;
            }
        }
        *n_comp = total;
        CLEAN_HIP(hipStreamSynchronize(s));
    } catch (const std::bad_alloc&) {
        return fail(SWV_ENOMEM, "swv_wavelet_clean: host allocation failed");
    }
    clear_error();
    return SWV_OK;
}
