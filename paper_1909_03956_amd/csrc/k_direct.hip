// Direct component sum (section 3.3, Eq. 12) on gfx950: the component
// ingest and the single-instance kernels.  Rows of a block are strided by
// the block size so each of a lane's VPL loads is coalesced.
#include <cmath>

#include "chunking.h"
#include "direct_rows.h"

namespace swv {

__global__ void k_ingest(int64_t n, const double* __restrict__ l, const double* __restrict__ m,
                         const double* __restrict__ flux, Comp* __restrict__ out,
                         int* __restrict__ status) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int bad;
    out[k] = pack_component(l[k], m[k], flux[k], bad);
    if (bad) atomicOr(status, bad);
}

__global__ void k_ingest_cell(int64_t n, const double* __restrict__ l,
                              const double* __restrict__ m, const double* __restrict__ flux,
                              CompCell* __restrict__ out, int* __restrict__ status) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int bad;
    out[k] = pack_component_cell(l[k], m[k], flux[k], bad);
    if (bad) atomicOr(status, bad);
}

hipError_t launch_ingest(hipStream_t s, int64_t n, const double* l, const double* m,
                         const double* flux, Comp* out, int* status) {
    if (n <= 0) return hipSuccess;
    const int b = 256;
    k_ingest<<<dim3((unsigned)((n + b - 1) / b)), dim3(b), 0, s>>>(n, l, m, flux, out, status);
    return hipGetLastError();
}

__global__ void k_ingest_f32c(int64_t n, const double* __restrict__ l,
                              const double* __restrict__ m, const double* __restrict__ flux,
                              CompF* __restrict__ out, int* __restrict__ status) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    int bad;
    out[k] = pack_component_f32c(l[k], m[k], flux[k], bad);
    if (bad) atomicOr(status, bad);
}

hipError_t launch_ingest(hipStream_t s, int64_t n, const double* l, const double* m,
                         const double* flux, CompF* out, int* status) {
    if (n <= 0) return hipSuccess;
    const int b = 256;
    k_ingest_f32c<<<dim3((unsigned)((n + b - 1) / b)), dim3(b), 0, s>>>(n, l, m, flux, out,
                                                                        status);
    return hipGetLastError();
}

hipError_t launch_ingest(hipStream_t s, int64_t n, const double* l, const double* m,
                         const double* flux, CompCell* out, int* status) {
    if (n <= 0) return hipSuccess;
    const int b = 256;
    k_ingest_cell<<<dim3((unsigned)((n + b - 1) / b)), dim3(b), 0, s>>>(n, l, m, flux, out,
                                                                        status);
    return hipGetLastError();
}

// ------------------------------------------------- FP64, few components ---
// Each block packs the components itself (one launch instead of two and no
// workspace: the call is latency-bound); lanes read them as LDS broadcasts.
// Two rows per lane from 3 x 2^20 rows on: fewer packings, and more row loads in
// flight where the call is bound by them.  15 components, one, two and four rows
// per lane: 2,000,000 rows 30.5, 31.9 and 32.9 us, 4,000,000 rows 60.5, 57.7 and
// 59.4, 10,000,000 rows 158, 153 and 155.
constexpr int kFewBlock = 256;

template <int VPL>
__global__ __launch_bounds__(kFewBlock) void k_direct_few(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    int64_t n_vis, const double* __restrict__ l, const double* __restrict__ m,
    const double* __restrict__ flux, int n_comp, double sgn, double2* __restrict__ out,
    int* __restrict__ status) {
    __shared__ Comp comp[kTableMinComp];
    if ((int)threadIdx.x < n_comp) {
        int bad;
        comp[threadIdx.x] = pack_component(l[threadIdx.x], m[threadIdx.x], flux[threadIdx.x], bad);
        if (bad && blockIdx.x == 0) atomicOr(status, bad);
    }
    __syncthreads();
    int64_t j[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i)
        j[i] = ((int64_t)blockIdx.x * VPL + i) * kFewBlock + threadIdx.x;
    const auto put = [out](int64_t row, double re, double im) { store_vis(out, row, re, im); };
    direct_rows_f64<VPL>(j, n_vis, u, v, w, (const Comp*)comp, n_comp, sgn, put, status);
}

// The same of packed components (a tree's leaf sum): scalar loads.
template <int VPL, class OUT>
__global__ __launch_bounds__(kFewBlock) void k_direct_few_packed(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    int64_t n_vis, const CompCell* __restrict__ comp, int n_comp, double sgn,
    OUT* __restrict__ out, int* __restrict__ status) {
    int64_t j[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i)
        j[i] = ((int64_t)blockIdx.x * VPL + i) * kFewBlock + threadIdx.x;
    const auto put = [out](int64_t row, double re, double im) { store_vis(out, row, re, im); };
    direct_rows_f64<VPL>(j, n_vis, u, v, w, uniform_ptr(comp), n_comp, sgn, put, status);
}

static int few_vpl(int64_t n_vis) { return n_vis < (int64_t(3) << 20) ? 1 : 2; }
static dim3 few_grid(int64_t n_vis) {
    const int64_t rows = kFewBlock * few_vpl(n_vis);
    return dim3((unsigned)((n_vis + rows - 1) / rows));
}

hipError_t launch_direct_few(hipStream_t s, int64_t n_vis, const double* u, const double* v,
                             const double* w, int n_comp, const double* l, const double* m,
                             const double* flux, int sign, double2* out, int* status) {
    if (n_comp >= kTableMinComp) return hipErrorInvalidValue;
    return launch_row_slabs(n_vis, [&](int64_t j, int64_t n) {
        const dim3 grid = few_grid(n), blk(kFewBlock);
        if (few_vpl(n) == 1)
            k_direct_few<1><<<grid, blk, 0, s>>>(u + j, v + j, w + j, n, l, m, flux, n_comp,
                                                 (double)sign, out + j, status);
        else
            k_direct_few<2><<<grid, blk, 0, s>>>(u + j, v + j, w + j, n, l, m, flux, n_comp,
                                                 (double)sign, out + j, status);
        return hipGetLastError();
    });
}

// -------------------------------------------------- FP64, table phasor ----
template <int VPL, class OUT>
__global__ __launch_bounds__(kTabBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_direct_cell(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    int64_t n_vis, const CompCell* __restrict__ comp, int n_comp, double sgn,
    OUT* __restrict__ out, int* __restrict__ status) {
    __shared__ Cell T[kTabCells];
    fill_cells(T);
    const int64_t base = (int64_t)blockIdx.x * (kTabBlock * VPL) + threadIdx.x;
    int64_t j[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) j[i] = base + (int64_t)i * kTabBlock;
    const auto put = [out](int64_t row, double re, double im) { store_vis(out, row, re, im); };
    direct_rows_cell<VPL>((CellPtr)T, j, n_vis, u, v, w, comp, n_comp, sgn, put, status);
}

// SPLIT waves of the workgroup share a row's components, 8 / SPLIT ranges each:
// calls too small to fill the chip by rows alone, and long component lists
// (direct_shape).  Their range sums meet in
// LDS (where the table was) and are added in range order.
template <int VPL, int SPLIT, class OUT>
__global__ __launch_bounds__(kTabBlock) __attribute__((amdgpu_waves_per_eu(4))) void
k_direct_cell_split(const double* __restrict__ u, const double* __restrict__ v,
                    const double* __restrict__ w, int64_t n_vis,
                    const CompCell* __restrict__ comp, int n_comp, double sgn,
                    OUT* __restrict__ out, int* __restrict__ status) {
    __shared__ Cell T[kTabCells];
    fill_cells(T);
    const auto put = [out](int64_t row, double re, double im) { store_vis(out, row, re, im); };
    direct_block_cell<VPL, SPLIT>(T, (int64_t)blockIdx.x * (kTabBlock / SPLIT * VPL), n_vis, u, v,
                                  w, comp, n_comp, sgn, put, status);
}

// The smallest row counts: workgroup (x, b) takes 64 rows and sub-range b of
// all 8 ranges, one range per wave; partial[a][b][row].
__global__ __launch_bounds__(kTabBlock) __attribute__((amdgpu_waves_per_eu(4))) void
k_direct_cell_part(const double* __restrict__ u, const double* __restrict__ v,
                   const double* __restrict__ w, int64_t n_vis,
                   const CompCell* __restrict__ comp, int n_comp, double2* __restrict__ partial,
                   int* __restrict__ status) {
    __shared__ Cell T[kTabCells];
    fill_cells(T);
    const int lane = threadIdx.x & 63, a = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.y;
    const int64_t j[1] = {(int64_t)blockIdx.x * 64 + lane};
    double U[1], V[1], W[1], re[1] = {0.0}, im[1] = {0.0};
    const bool wide = load_rows<1>(j, n_vis, u, v, w, U, V, W);
    const CompRanges R(n_comp);
    const int k0 = R.begin(a, b), k1 = R.end(a, b);
    if (__builtin_expect(wide, 0))
        add_components<1, true>((CellPtr)T, uniform_ptr(comp), k0, k1, U, V, W, re, im);
    else
        add_components<1, false>((CellPtr)T, uniform_ptr(comp), k0, k1, U, V, W, re, im);
    if (j[0] < n_vis) {
        if (a == 0 && b == 0 && !isfinite(U[0] + V[0] + W[0])) atomicOr(status, kStatusNonFinite);
        partial[((int64_t)a * 8 + b) * n_vis + j[0]] = make_double2(re[0], im[0]);
    }
}

template <class OUT>
__global__ __launch_bounds__(64) void k_direct_join(const double2* __restrict__ partial,
                                                    int64_t n_vis, double sgn,
                                                    OUT* __restrict__ out) {
    const int64_t j = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (j >= n_vis) return;
    double re = 0.0, im = 0.0;
#pragma unroll
    for (int a = 0; a < 8; ++a) {
        double rr = 0.0, ri = 0.0;
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const double2 p = partial[((int64_t)a * 8 + b) * n_vis + j];
            rr += p.x;
            ri += p.y;
        }
        re += rr;
        im += ri;
    }
    store_vis(out, j, re, sgn * im);
}

// Layout with the least estimated time.  A workgroup's time, in units of one
// wave's (64 rows, component) pass with the CU full (two workgroups): per_comp x
// components of a wave (fewer rows per lane cost a little more each, for the
// per-component copies and loads), plus about 14 for filling the table.  Shared by
// waves, a row's components make more and shorter workgroups, which even out over
// the dies' different clocks: 4 rows a lane over 1, 4 and 8 waves take 8.63, 8.30
// and 8.17 ms (8,355,840 rows x 2,000 components), 1.28, 1.22 and 1.25 ms
// (8,000,000 x 300) and 0.143, 0.159 and 0.180 ms (4,000,000 x 60).
// Workgroups run in rounds of two per CU; a call of one workgroup per CU or less
// gets no credit for that, since nothing keeps two of them off the same CU
// (261,120 rows x 1,000 components in 255 workgroups: 180 us at best, 336 us
// behind the ingest kernel).
DirectShape direct_shape(int64_t n_vis, int64_t n_comp, int vpl_max, int n_cu, bool partials) {
    const struct {
        int vpl, split, parts;
        double per_comp;
    } all[] = {{4, 1, 1, 4.0}, {4, 4, 1, 3.85}, {4, 8, 1, 3.75}, {2, 1, 1, 2.04}, {1, 1, 1, 1.28}, {2, 2, 1, 2.04}, {2, 4, 1, 2.04},
               {1, 2, 1, 1.28}, {1, 4, 1, 1.28}, {1, 8, 1, 1.28}, {1, 8, 8, 1.28}};
    DirectShape best;
    double best_t = HUGE_VAL;
    for (const auto& c : all) {
        if (c.vpl > vpl_max) continue;
        const int64_t rows = (int64_t)kTabBlock / c.split * c.vpl;
        const int64_t blocks = (n_vis + rows - 1) / rows * c.parts;
        // the partial sums of a call cost a second launch and 2 x 1 KB a row
        if (c.parts > 1 && (!partials || blocks > 4 * (int64_t)n_cu || n_comp < 256)) continue;
        const int64_t rounds = (blocks + 2 * (int64_t)n_cu - 1) / (2 * (int64_t)n_cu);
        double t = (double)rounds * (c.per_comp * (double)n_comp / (c.split * c.parts) + 14.0);
        if (c.parts > 1) t += 45.0;   // the second launch
        if (t < best_t) {
            best_t = t;
            best.vpl = c.vpl;
            best.split = c.split;
            best.parts = c.parts;
        }
    }
    return best;
}

template <class OUT>
static hipError_t run_direct_cell(hipStream_t s, const DirectShape& sh, int64_t n_vis,
                                  const double* u, const double* v, const double* w,
                                  const CompCell* comp, int64_t n_comp, int sign, OUT* out,
                                  double2* partial, int* status) {
    const double sg = (double)sign;
    const int nc = (int)n_comp;
    if (n_comp < kTableMinComp) {
        if (few_vpl(n_vis) == 1)
            k_direct_few_packed<1, OUT><<<few_grid(n_vis), dim3(kFewBlock), 0, s>>>(
                u, v, w, n_vis, comp, nc, sg, out, status);
        else
            k_direct_few_packed<2, OUT><<<few_grid(n_vis), dim3(kFewBlock), 0, s>>>(
                u, v, w, n_vis, comp, nc, sg, out, status);
        return hipGetLastError();
    }
    const dim3 blk(kTabBlock);
    const int64_t rows = (int64_t)kTabBlock / sh.split * sh.vpl;
    const unsigned nb = (unsigned)((n_vis + rows - 1) / rows);
    if (sh.parts > 1) {
        if (!partial || sh.split != 8 || sh.parts != 8) return hipErrorInvalidValue;
        k_direct_cell_part<<<dim3(nb, 8), blk, 0, s>>>(u, v, w, n_vis, comp, nc, partial, status);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        k_direct_join<OUT><<<dim3(nb), dim3(64), 0, s>>>(partial, n_vis, sg, out);
        return hipGetLastError();
    }
#define SWV_CELL(V, S) \
    if (sh.vpl == V && sh.split == S)
    SWV_CELL(4, 1) k_direct_cell<4, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(2, 1) k_direct_cell<2, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(1, 1) k_direct_cell<1, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(2, 2) k_direct_cell_split<2, 2, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(2, 4) k_direct_cell_split<2, 4, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(4, 4) k_direct_cell_split<4, 4, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(4, 8) k_direct_cell_split<4, 8, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(1, 2) k_direct_cell_split<1, 2, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(1, 4) k_direct_cell_split<1, 4, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else SWV_CELL(1, 8) k_direct_cell_split<1, 8, OUT><<<dim3(nb), blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status);
    else return hipErrorInvalidValue;
#undef SWV_CELL
    return hipGetLastError();
}

hipError_t launch_direct_cell(hipStream_t s, const DirectShape& sh, int64_t n_vis, const double* u,
                              const double* v, const double* w, const CompCell* comp,
                              int64_t n_comp, int sign, int prec, void* out, double2* partial,
                              int* status) {
    return launch_row_slabs(n_vis, [&](int64_t j, int64_t n) {
        if (prec == SWV_FP64)
            return run_direct_cell(s, sh, n, u + j, v + j, w + j, comp, n_comp, sign,
                                   (double2*)out + j, partial, status);
        return run_direct_cell(s, sh, n, u + j, v + j, w + j, comp, n_comp, sign,
                               (float2*)out + j, partial, status);
    });
}

// ------------------------------------------------------------------ F32C ---
template <int VPL, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_direct_f32c(const double* __restrict__ u,
                                                       const double* __restrict__ v,
                                                       const double* __restrict__ w,
                                                       int64_t n_vis,
                                                       const CompF* __restrict__ comp, int n_comp,
                                                       double sgn, float2* __restrict__ out,
                                                       int* __restrict__ status) {
    const int64_t base = (int64_t)blockIdx.x * (BLOCK * VPL) + threadIdx.x;
    int64_t j[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) j[i] = base + (int64_t)i * BLOCK;
    direct_rows_f32c<VPL>(j, n_vis, u, v, w, comp, n_comp, sgn, out, status);
}

// Calls too small to fill the chip by rows alone: SPLIT waves of the workgroup
// share a row's components, every SPLIT-th range each; the range sums meet in LDS.
constexpr int kF32cBlock = 512;

template <int SPLIT>
__global__ __launch_bounds__(kF32cBlock) void k_direct_f32c_split(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    int64_t n_vis, const CompF* __restrict__ comp, int n_comp, double sgn,
    float2* __restrict__ out, int* __restrict__ status) {
    constexpr int kRows = kF32cBlock / SPLIT;
    __shared__ double2 part[8][kRows];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int own = wave % SPLIT, local = wave / SPLIT * 64 + lane;
    const int64_t row0 = (int64_t)blockIdx.x * kRows;
    const int64_t j[1] = {row0 + local};
    double U[1], V[1], W[1];
    load_rows_f32c<1>(j, n_vis, u, v, w, U, V, W);
    const CompRanges R(n_comp, kF32cSub, kF32cRange);
    const auto keep = [&](int a, const double(&re)[1], const double(&im)[1]) {
        part[a][local] = make_double2(re[0], im[0]);
    };
#pragma unroll 1
    for (int a = own; a < 8; a += SPLIT)
        range_sums_f32c<1>(uniform_ptr(comp), R, a, a + 1, U, V, W, keep);
    __syncthreads();
    for (int r = threadIdx.x; r < kRows && row0 + r < n_vis; r += kF32cBlock) {
        double re = 0.0, im = 0.0;
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            re += part[a][r].x;
            im += part[a][r].y;
        }
        const int64_t jr = row0 + r;
        if (!isfinite(u[jr] + v[jr] + w[jr])) atomicOr(status, kStatusNonFinite);
        store_vis(out, jr, re, sgn * im);
    }
}

// The smallest row counts: workgroup (x, b) takes 64 rows and sub-range b of all
// 8 ranges, one range per wave; partial[a][b][row], joined as in FP64.
__global__ __launch_bounds__(kF32cBlock) void k_direct_f32c_part(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    int64_t n_vis, const CompF* __restrict__ comp, int n_comp, double2* __restrict__ partial,
    int* __restrict__ status) {
    const int lane = threadIdx.x & 63, a = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = blockIdx.y;
    const int64_t j[1] = {(int64_t)blockIdx.x * 64 + lane};
    double U[1], V[1], W[1], re[1] = {0.0}, im[1] = {0.0};
    load_rows_f32c<1>(j, n_vis, u, v, w, U, V, W);
    const CompRanges R(n_comp, kF32cSub, kF32cRange);
    const int k0 = R.begin(a, b), k1 = R.end(a, b);
    add_components_f32c<1>(uniform_ptr(comp), k0, k1, U, V, W, re, im);
    if (j[0] < n_vis) {
        if (a == 0 && b == 0 && !isfinite(U[0] + V[0] + W[0])) atomicOr(status, kStatusNonFinite);
        partial[((int64_t)a * 8 + b) * n_vis + j[0]] = make_double2(re[0], im[0]);
    }
}

// A wave alone on its SIMD runs at its latencies: components are shared until
// there are 4 waves for each of them, by the workgroups too where the ranges have
// sub-ranges enough to pay for the second launch.
DirectShape direct_shape_f32c(int64_t n_vis, int64_t n_comp, int n_cu, bool partials) {
    const int64_t waves = (n_vis + 63) / 64, want = 16 * (int64_t)n_cu;
    DirectShape sh;
    while (sh.split < 8 && waves * sh.split < want && n_comp >= kF32cRange * sh.split) sh.split *= 2;
    if (partials && sh.split == 8 && waves * 8 * 2 <= want && n_comp >= 32 * kF32cSub) sh.parts = 8;
    return sh;
}

template <int VPL, int BLOCK>
static hipError_t run_direct(hipStream_t s, int64_t n_vis, const double* u, const double* v,
                             const double* w, const CompF* comp, int64_t n_comp, int sign,
                             void* out, int* status) {
    const int64_t rows = (int64_t)BLOCK * VPL;
    const dim3 grid((unsigned)((n_vis + rows - 1) / rows)), blk(BLOCK);
    k_direct_f32c<VPL, BLOCK><<<grid, blk, 0, s>>>(u, v, w, n_vis, comp, (int)n_comp, (double)sign,
                                                   (float2*)out, status);
    return hipGetLastError();
}

template <int VPL>
static hipError_t run_direct_b(hipStream_t s, int block, int64_t n_vis, const double* u,
                               const double* v, const double* w, const CompF* comp, int64_t n_comp,
                               int sign, void* out, int* status) {
    switch (block) {
        case 64: return run_direct<VPL, 64>(s, n_vis, u, v, w, comp, n_comp, sign, out, status);
        case 128: return run_direct<VPL, 128>(s, n_vis, u, v, w, comp, n_comp, sign, out, status);
        case 256: return run_direct<VPL, 256>(s, n_vis, u, v, w, comp, n_comp, sign, out, status);
        default: return hipErrorInvalidValue;
    }
}

static hipError_t run_direct_f32c(hipStream_t s, const DirectShape& sh, int vpl, int block,
                                  int64_t n_vis, const double* u, const double* v,
                                  const double* w, const CompF* comp, int64_t n_comp, int sign,
                                  float2* out, double2* partial, int* status) {
    const int nc = (int)n_comp;
    const double sg = (double)sign;
    if (sh.parts > 1) {
        if (!partial || sh.split != 8 || sh.parts != 8) return hipErrorInvalidValue;
        const unsigned nb = (unsigned)((n_vis + 63) / 64);
        k_direct_f32c_part<<<dim3(nb, 8), dim3(kF32cBlock), 0, s>>>(u, v, w, n_vis, comp, nc,
                                                                    partial, status);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        k_direct_join<float2><<<dim3(nb), dim3(64), 0, s>>>(partial, n_vis, sg, out);
        return hipGetLastError();
    }
    if (sh.split > 1) {
        const int64_t rows = kF32cBlock / sh.split;
        const dim3 grid((unsigned)((n_vis + rows - 1) / rows)), blk(kF32cBlock);
        switch (sh.split) {
            case 2: k_direct_f32c_split<2><<<grid, blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status); break;
            case 4: k_direct_f32c_split<4><<<grid, blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status); break;
            case 8: k_direct_f32c_split<8><<<grid, blk, 0, s>>>(u, v, w, n_vis, comp, nc, sg, out, status); break;
            default: return hipErrorInvalidValue;
        }
        return hipGetLastError();
    }
    switch (vpl) {
        case 1: return run_direct_b<1>(s, block, n_vis, u, v, w, comp, n_comp, sign, out, status);
        case 2: return run_direct_b<2>(s, block, n_vis, u, v, w, comp, n_comp, sign, out, status);
        case 4: return run_direct_b<4>(s, block, n_vis, u, v, w, comp, n_comp, sign, out, status);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_direct_f32c(hipStream_t s, const DirectShape& sh, int vpl, int block,
                              int64_t n_vis, const double* u, const double* v, const double* w,
                              const CompF* comp, int64_t n_comp, int sign, void* out,
                              double2* partial, int* status) {
    return launch_row_slabs(n_vis, [&](int64_t j, int64_t n) {
        return run_direct_f32c(s, sh, vpl, block, n, u + j, v + j, w + j, comp, n_comp, sign,
                               (float2*)out + j, partial, status);
    });
}

}  // namespace swv
