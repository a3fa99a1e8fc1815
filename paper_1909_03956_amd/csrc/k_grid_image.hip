// Exact dirty images on a regular grid (section 2.2):
//     img(x, y) = Re sum_j exp(-s 2 pi i (u l_x + v m_y + w (n_xy - 1))) y_j
// with the phasor split over the grid's axes.  For a row,
//     exp(i phi) = E_x(l) E_y(m) E_w(n - 1),
// E_x and E_y depend on one coordinate each and n - 1 only on (l^2, m^2), so
// the four pixels (+-l, +-m) share E_w, and with z = E_w y (y conjugated for
// s = +1) their real parts are signed sums of four products:
//     img(sl l, sm m) = P - sl sm Q - sl R - sm S,
//     P = sum zr cx cy,  Q = sum zr sx sy,  R = sum zi sx cy,  S = sum zi cx sy.
// The kernel accumulates P, Q, R, S per quad (|l|, |m|): 25 FP64 instructions
// per row and quad (4 for the w phase and its cell, 5 for the rest of the
// angle, 8 to turn y, 8 for the products), 6.25 a pixel where the general
// adjoint takes 20 (table phasor) and throws its imaginary half away.  n - 1 is
// also the same for (|l|, |m|) and (|m|, |l|): such a pair of quads, an octet,
// shares z and takes 33.  Bound by FP64 issue: 176,904 rows x 256^2 pixels
// 2.64 ms (19.6 by the adjoint with the polynomial phasor, 2.90 by quads alone),
// 88,904 rows of a 511^2 beam (y = 1, four instructions less) 4.60 ms (30; 5.10).
//
// Accuracy: the phases u l, v m are reduced with their products' rounding
// errors, w (n - 1) enters the cell search and the rest by FMAs, so no phase is
// rounded at its own magnitude; each phasor is good to a few 2^-53.
//
// Layout.  A prep kernel writes, for a slab of rows, {w, y} records and the
// tables E_x, E_y (16 (Kx + Ky) + 32 bytes a row; slabs bound the workspace).
// A wave takes 64 neighbouring |k| of one axis (the lane axis, E by coalesced
// vector loads) and a few of the other (E by scalar loads, an SGPR operand of
// every lane's products).  The square of whole 64 x 64 blocks goes by octets below
// its diagonal and by quads on it.  Kx is rarely a multiple of 64 (129 for a
// 256-pixel side): what is left over beyond whole waves is covered by strips with
// the axes exchanged.
//
// Jobs (wave, chunk of rows) are numbered chunk-major and dealt in runs, one run
// of workgroups per XCD, as in the adjoint.
#include <type_traits>

#include "chunking.h"
#include "device_math.h"
#include "launch.h"
#include "phasor_table.h"

namespace swv {

namespace {

constexpr int kStep = 4;   // scalar-axis positions per wave of quads
constexpr int kOct = 2;    // of octets

// One row of a slab as the kernel reads it (scalar loads); wide: |w| asks for
// the WIDE form of the cell search.
struct alignas(32) GridRow {
    double w, yr, yi;
    long long wide;
};

// (cos, sin)(2 pi u k cell) of one row and grid offset k, the product's rounding
// error kept.
__device__ __forceinline__ Cell axis_phasor(double u, double x) {
    const double p = u * x;
    double r = (p - rint(p)) + fma(u, x, -p);
    r -= rint(r);
    double c, q;
    cis2pi_q(r, c, q);
    return Cell{c, 4.0 * q};
}

}  // namespace

// Thread (row, position): E_x for positions below Kx, then E_y; the first
// thread of a row also writes its record.
__global__ __launch_bounds__(256) void k_grid_prep(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    const double2* __restrict__ y, int64_t n, GridGeom g, double ysign, GridRow* __restrict__ rec,
    Cell* __restrict__ ex, Cell* __restrict__ ey) {
    const int K = g.Kx + g.Ky;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n * K; i += stride) {
        const int64_t j = i / K;
        const int k = (int)(i - j * K);
        if (k < g.Kx)
            ex[j * g.Kx + k] = axis_phasor(u[j], (double)(g.kx0 + k) * g.cell);
        else
            ey[j * g.Ky + (k - g.Kx)] = axis_phasor(v[j], (double)(g.ky0 + k - g.Kx) * g.cell);
        if (k == 0) {
            const double2 a = y ? y[j] : make_double2(1.0, 0.0);
            rec[j] = GridRow{w[j], a.x, ysign * a.y, fabs(w[j]) < kTabMaxBaseline ? 0 : 1};
        }
    }
}

namespace {

using RowPtr = const __attribute__((address_space(4))) GridRow*;
using ScalarCells = const __attribute__((address_space(4))) Cell*;

// (zr, zi) of G phases w nm1[i]: E_w y, UNIT for y = 1.
template <int G, bool UNIT, bool WIDE>
__device__ __forceinline__ void turn_row_value(CellPtr T, const CellCoefs& K, double w, double yr,
                                               double yi, const double (&nm1)[G], double (&zr)[G],
                                               double (&zi)[G]) {
    Cell e[G];
    double d[G];
#pragma unroll
    for (int i = 0; i < G; ++i) e[i] = find_cell_product<WIDE>(T, w, nm1[i], K.magic, d[i]);
#pragma unroll
    for (int i = 0; i < G; ++i) {
        double cr, sr;
        cell_rest(K, d[i], cr, sr);
        double tr = cr, ti = sr;
        if constexpr (!UNIT) {
            tr = fma(cr, yr, -(sr * yi));
            ti = fma(cr, yi, sr * yr);
        }
        zr[i] = fma(e[i].x, tr, -(e[i].y * ti));
        zi[i] = fma(e[i].x, ti, e[i].y * tr);
    }
}

// acc += (P, Q, R, S) of one quad: a the lane axis' phasor, b the step axis' (R
// has the lane axis' sine).
__device__ __forceinline__ void add_quad(double zr, double zi, Cell a, double cb, double sb,
                                         double (&acc)[4]) {
    acc[0] = fma(zr * a.x, cb, acc[0]);
    acc[1] = fma(zr * a.y, sb, acc[1]);
    acc[2] = fma(zi * a.y, cb, acc[2]);
    acc[3] = fma(zi * a.x, sb, acc[3]);
}

// Rows of a chunk into Q quads per lane and step position: Q = 1, or 2 for octets,
// whose second quad has the other axis' tables at the same positions.
template <int G, int Q, bool UNIT, bool WIDE>
__device__ __forceinline__ void add_rows(CellPtr T, RowPtr R, int nrow,
                                         const Cell* __restrict__ A, int KA, ScalarCells B, int KB,
                                         const Cell* __restrict__ A2, ScalarCells B2,
                                         const double (&nm1)[G], double (&acc)[Q][G][4]) {
    const CellCoefs K = cell_coefs();
    Cell next = A[0], next2 = Q == 2 ? A2[0] : Cell{0.0, 0.0};
#pragma unroll 1
    for (int j = 0; j < nrow; ++j) {
        const Cell a = next, a2 = next2;
        const int64_t jn = j + 1 < nrow ? j + 1 : j;   // ahead of this row's arithmetic
        next = A[jn * KA];
        if constexpr (Q == 2) next2 = A2[jn * KB];
        double zr[G], zi[G];
        turn_row_value<G, UNIT, WIDE>(T, K, R[j].w, R[j].yr, R[j].yi, nm1, zr, zi);
        const ScalarCells b = B + (int64_t)j * KB;
#pragma unroll
        for (int i = 0; i < G; ++i) add_quad(zr[i], zi[i], a, b[i].x, b[i].y, acc[0][i]);
        if constexpr (Q == 2) {
            const ScalarCells b2 = B2 + (int64_t)j * KA;
#pragma unroll
            for (int i = 0; i < G; ++i) add_quad(zr[i], zi[i], a2, b2[i].x, b2[i].y, acc[1][i]);
        }
    }
}

struct GridData {
    const GridRow* rec;
    const Cell *ex, *ey;
    double* partial;
    bool resume;
};

// One wave's quads or octets (lane position `lane`, step positions step ..
// step + G) over the rows of a chunk.
template <int G, int Q, bool UNIT>
__device__ __forceinline__ void grid_wave(CellPtr T, const GridGeom& g, bool swapped, int lane,
                                          int lane_end, int step, int step_end, int64_t j0,
                                          int nrow, bool wide, const GridData& data,
                                          int64_t quad_base) {
    const int la = lane < lane_end ? lane : lane_end - 1;   // idle lanes repeat the last
    const int KA = swapped ? g.Ky : g.Kx, KB = swapped ? g.Kx : g.Ky;
    const Cell* __restrict__ A = (swapped ? data.ey : data.ex) + j0 * KA + la;
    const ScalarCells B = uniform_ptr((swapped ? data.ex : data.ey) + j0 * KB + step);
    // octets (lanes along x): the other quad's lane axis is y, its step axis x
    const Cell* __restrict__ A2 = data.ey + j0 * KB + la;
    const ScalarCells B2 = uniform_ptr(data.ex + j0 * KA + step);
    const RowPtr R = uniform_ptr(data.rec + j0);
    double nm1[G], acc[Q][G][4];
    int64_t quad[Q][G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int st = step + i < step_end ? step + i : step_end - 1;
        const int kx = swapped ? st : la, ky = swapped ? la : st;
        nm1[i] = g.nm1(kx, ky);
        quad[0][i] = quad_base + (int64_t)ky * g.Kx + kx;
        if constexpr (Q == 2) quad[1][i] = quad_base + (int64_t)kx * g.Kx + ky;
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                // lanes along y: R and S change places
                const int at = (swapped || q == 1) && t >= 2 ? 5 - t : t;
                acc[q][i][t] = data.resume ? data.partial[4 * quad[q][i] + at] : 0.0;
            }
    }
    if (__builtin_expect(wide, 0))
        add_rows<G, Q, UNIT, true>(T, R, nrow, A, KA, B, KB, A2, B2, nm1, acc);
    else
        add_rows<G, Q, UNIT, false>(T, R, nrow, A, KA, B, KB, A2, B2, nm1, acc);
#pragma unroll
    for (int i = 0; i < G; ++i)
        if (lane < lane_end && step + i < step_end)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                double2* o = (double2*)(data.partial + 4 * quad[q][i]);
                const double(&x)[4] = acc[q][i];
                o[0] = make_double2(x[0], x[1]);
                o[1] = swapped || q == 1 ? make_double2(x[3], x[2]) : make_double2(x[2], x[3]);
            }
}

}  // namespace

namespace {

// Region, lane position and first step of a job of the regions, `step` positions
// to a job; lane tiles run fastest, so neighbouring waves share their positions.
__device__ __forceinline__ GridRegion region_job(const GridPlan& p, int64_t job, int per, int lane,
                                                 int& la, int& step) {
    int q = 0;
    while (q < 2 && job >= p.region_jobs[q]) job -= p.region_jobs[q++];
    const GridRegion r = p.region[q];
    const int lt = (r.lane_n + 63) / 64;
    la = r.lane0 + (int)(job % lt) * 64 + lane;
    step = r.step0 + (int)(job / lt) * per;
    return r;
}

}  // namespace

template <bool UNIT>
__global__ __launch_bounds__(kTabBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_grid_sums(
    GridGeom g, GridPlan p, int64_t n_rows, int64_t chunk, int64_t jobs, int64_t run,
    GridData data) {
    __shared__ Cell T[kTabCells];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t bid = blockIdx.x;
    const int64_t all = ((bid & 7) * run + (bid >> 3)) * (kTabBlock / 64) + wave;
    fill_cells(T);
    if (all >= jobs) return;
    const int64_t chunk_id = all / p.jobs;
    int64_t job = all - chunk_id * p.jobs;
    const int64_t j0 = chunk_id * chunk;
    const int nrow = __builtin_amdgcn_readfirstlane(
        (int)(j0 + chunk < n_rows ? chunk : n_rows - j0));
    const int64_t base = chunk_id * (int64_t)g.Kx * g.Ky;
    const CellPtr TP = (CellPtr)T;
    // a row that needs the WIDE form puts the whole chunk through it
    bool any = false;
    for (int j = lane; j < nrow; j += 64) any = any || data.rec[j0 + j].wide != 0;
    const bool wide = __any(any);
    if (job < p.oct_jobs) {
        // block row b of the square has 64 b / kOct jobs, the ones above it 16 b (b - 1)
        static_assert(kOct == 2, "numbering of the octets");
        int b = (int)((1.0f + sqrtf(1.0f + 0.25f * (float)job)) * 0.5f);
        while (16 * (int64_t)b * (b - 1) > job) --b;
        while (16 * (int64_t)(b + 1) * b <= job) ++b;
        b = __builtin_amdgcn_readfirstlane(b);
        const int step =
            __builtin_amdgcn_readfirstlane((int)(job - 16 * (int64_t)b * (b - 1)) * kOct);
        grid_wave<kOct, 2, UNIT>(TP, g, false, 64 * b + lane, 64 * b + 64, step, 64 * b, j0, nrow,
                                 wide, data, base);
        return;
    }
    job -= p.oct_jobs;
    GridRegion r;
    int la, step;
    if (job < p.diag_jobs) {
        const int b = (int)(job / (64 / kStep));
        r = GridRegion{64 * b, 64, 64 * b, 64, false};
        la = 64 * b + lane;
        step = 64 * b + (int)(job % (64 / kStep)) * kStep;
    } else {
        r = region_job(p, job - p.diag_jobs, kStep, lane, la, step);
    }
    step = __builtin_amdgcn_readfirstlane(step);
    const int lane_end = r.lane0 + r.lane_n, step_end = r.step0 + r.step_n;
    const int left = __builtin_amdgcn_readfirstlane(step_end - step);
    if (left > 2)
        grid_wave<4, 1, UNIT>(TP, g, r.swapped, la, lane_end, step, step_end, j0, nrow, wide, data,
                              base);
    else if (left == 2)
        grid_wave<2, 1, UNIT>(TP, g, r.swapped, la, lane_end, step, step_end, j0, nrow, wide, data,
                              base);
    else
        grid_wave<1, 1, UNIT>(TP, g, r.swapped, la, lane_end, step, step_end, j0, nrow, wide, data,
                              base);
}

// ------------------------------------------------------- FP32-compensated ---
// The same pixels by four in the FP32-compensated adjoint's arithmetic: phases,
// FP32 phasors, products in row pairs, Kahan steps and chunks are the adjoint's, so
// the sums' bits are its real parts'.  What the form saves: the imaginary half (a
// row costs a pixel 3.5 FP32 instructions instead of 7) and, of the phase's three
// FP64 ones, w (n - 1) is shared by the four pixels and v m by two: 1.75.  Bound by
// issue, the hardware sine and cosine the most of it.  176,904 rows x 256^2 pixels:
// 4.63 -> 3.94 ms (4.10 in 256-thread workgroups), 88,904 rows of a 511^2 beam 9.19
// -> 6.74 ms.
constexpr int kF32Block = 64;   // waves of a workgroup share nothing
constexpr int kF32Step = 2;   // quads per lane

namespace {

template <int G, bool UNIT>
__device__ __forceinline__ void image_f32c_rows(const double* u, const double* v, const double* w,
                                                const double2* y, int nrow, float fsg,
                                                const double (&l)[G], const double (&m)[G],
                                                const double (&nm1)[G], float (&sum)[G][4],
                                                float (&comp)[G][4]) {
    const auto* U = uniform_ptr(u);
    const auto* V = uniform_ptr(v);
    const auto* W = uniform_ptr(w);
    const auto* Y = uniform_ptr(y);
    const auto step = [&](auto count, int j) {
        constexpr int N = decltype(count)::value;
        float yr[N], yi[N];
#pragma unroll
        for (int r = 0; r < N; ++r) {
            yr[r] = UNIT ? 1.0f : (float)Y[j + r].x;
            yi[r] = UNIT ? 0.0f : fsg * (float)Y[j + r].y;
        }
#pragma unroll
        for (int i = 0; i < G; ++i) {
            float acc[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = -comp[i][t];
#pragma unroll
            for (int r = N - 1; r >= 0; --r) {
                const double wn = W[j + r] * nm1[i];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    // pixel (sl, sm) = (+-, +-): sl < 0 for odd t, sm < 0 for t >= 2
                    const double inner = fma(V[j + r], t & 2 ? -m[i] : m[i], wn);
                    const double ph = fma(U[j + r], t & 1 ? -l[i] : l[i], inner);
                    float c, s;
                    cis2pi_f32((float)__builtin_amdgcn_fract(ph), c, s);
                    if constexpr (!UNIT) acc[t] = fmaf(s, yi[r], acc[t]);
                    acc[t] = fmaf(c, yr[r], acc[t]);
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) kahan_step(acc[t], sum[i][t], comp[i][t]);
        }
    };
    int j = 0;
#pragma unroll 1
    for (; j + 2 <= nrow; j += 2) step(std::integral_constant<int, 2>(), j);
    if (j < nrow) step(std::integral_constant<int, 1>(), j);
}

template <int G, bool UNIT>
__device__ __forceinline__ void image_f32c_wave(const GridGeom& g, const GridRegion& r, int lane,
                                                int step, const double* u, const double* v,
                                                const double* w, const double2* y, int nrow,
                                                float fsg, double* partial) {
    const int lane_end = r.lane0 + r.lane_n, la = lane < lane_end ? lane : lane_end - 1;
    double l[G], m[G], nm1[G];
    float sum[G][4], comp[G][4];
    int64_t quad[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int kx = r.swapped ? step + i : la, ky = r.swapped ? la : step + i;
        quad[i] = (int64_t)ky * g.Kx + kx;
        nm1[i] = g.nm1(kx, ky);
        l[i] = (double)(g.kx0 + kx) * g.cell;
        m[i] = (double)(g.ky0 + ky) * g.cell;
#pragma unroll
        for (int t = 0; t < 4; ++t) sum[i][t] = comp[i][t] = 0.0f;
    }
    image_f32c_rows<G, UNIT>(u, v, w, y, nrow, fsg, l, m, nm1, sum, comp);
#pragma unroll
    for (int i = 0; i < G; ++i)
        if (lane < lane_end) {
            double x[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) x[t] = (double)sum[i][t] - (double)comp[i][t];
            double2* o = (double2*)(partial + 4 * quad[i]);
            o[0] = make_double2(x[0], x[1]);
            o[1] = make_double2(x[2], x[3]);
        }
}

}  // namespace

template <bool UNIT>
__global__ __launch_bounds__(kF32Block) void k_image_f32c(
    GridGeom g, GridPlan p, const double* __restrict__ u, const double* __restrict__ v,
    const double* __restrict__ w, const double2* __restrict__ y, int64_t n_vis, int64_t chunk,
    int64_t jobs, int64_t run, float fsg, double* __restrict__ partial) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t bid = blockIdx.x;
    const int64_t all = ((bid & 7) * run + (bid >> 3)) * (kF32Block / 64) + wave;
    if (all >= jobs) return;
    const int64_t chunk_id = all / p.jobs, j0 = chunk_id * chunk;
    const int nrow =
        __builtin_amdgcn_readfirstlane((int)(j0 + chunk < n_vis ? chunk : n_vis - j0));
    int la, step;
    const GridRegion r = region_job(p, all - chunk_id * p.jobs, p.step, lane, la, step);
    double* part = partial + chunk_id * 4 * (int64_t)g.Kx * g.Ky;
    const double2* yy = y ? y + j0 : nullptr;
    if (p.step >= 2 && __builtin_amdgcn_readfirstlane(r.step0 + r.step_n - step) >= 2)
        image_f32c_wave<2, UNIT>(g, r, la, step, u + j0, v + j0, w + j0, yy, nrow, fsg, part);
    else
        image_f32c_wave<1, UNIT>(g, r, la, step, u + j0, v + j0, w + j0, yy, nrow, fsg, part);
}

// Adds the chunks of each quad (16 threads take every 16th chunk in order, their
// sums meet in a fixed tree) and writes its pixels, 0 off the unit disk: from the
// sums P, Q, R, S, or (PIXELS) from one sum for each.
constexpr int kFinCols = 16, kFinQ = 16;

template <bool PIXELS>
__global__ __launch_bounds__(kFinCols * 4 * kFinQ) void k_grid_finish(
    GridGeom g, const double* __restrict__ partial, int64_t n_chunks, int64_t bid0, int nx, int ny,
    int cx, int cy, double n_vis, double* __restrict__ img) {
    __shared__ double red[kFinQ][kFinCols * 4];
    const int64_t quads = (int64_t)g.Kx * g.Ky;
    const int tx = threadIdx.x % (kFinCols * 4), r = threadIdx.x / (kFinCols * 4);
    const int64_t at = (bid0 + blockIdx.x) * (kFinCols * 4) + tx;   // 4 quad + component
    double s = 0.0;
    if (at < 4 * quads)
        for (int64_t c = r; c < n_chunks; c += kFinQ) s += partial[c * 4 * quads + at];
    red[r][tx] = s;
    __syncthreads();
    for (int h = kFinQ / 2; h > 0; h >>= 1) {
        if (r < h) red[r][tx] += red[r + h][tx];
        __syncthreads();
    }
    if (r != 0 || at >= 4 * quads) return;
    // thread t of a quad writes the pixel with signs (sl, sm)
    const double* q4 = &red[0][tx & ~3];
    const int sl = (tx & 1) ? -1 : 1, sm = (tx & 2) ? -1 : 1;
    const int64_t quad = at >> 2;
    const int ky = (int)(quad / g.Kx), kx = (int)(quad - (int64_t)ky * g.Kx);
    const int ax = g.kx0 + kx, ay = g.ky0 + ky;
    if ((sl < 0 && ax == 0) || (sm < 0 && ay == 0)) return;
    const int64_t ix = (int64_t)cx + (int64_t)sl * ax, iy = (int64_t)cy + (int64_t)sm * ay;
    if (ix < 0 || ix >= nx || iy < 0 || iy >= ny) return;
    const double v = PIXELS ? red[0][tx]
                            : (q4[0] - (sl * sm) * q4[1]) - (sl * q4[2] + sm * q4[3]);
    img[iy * nx + ix] = g.on_disk(kx, ky) ? v / n_vis : 0.0;
}

// ------------------------------------------------------------------- plan --
// Distinct |i - c| of i = 0 .. n - 1: `count` from `first`.
static void axis_offsets(int n, int64_t c, int64_t* first, int64_t* count) {
    const int64_t lo = -c, hi = (int64_t)n - 1 - c;
    const int64_t a = lo < 0 ? -lo : lo, b = hi < 0 ? -hi : hi;
    *first = lo <= 0 && hi >= 0 ? 0 : (a < b ? a : b);
    *count = (a > b ? a : b) - *first + 1;
}

// Instructions per row of a wave of `n` step positions.
static int64_t quads_cost(int64_t n) { return 25 * n; }

// Covers x in [x0, x0 + nX), y in [y0, y0 + nY) by at most two regions: lanes along
// the axis that wastes less, and its rest beyond whole waves either as one more,
// partly idle lane tile or as a strip with the axes exchanged.  Returns the cost.
static int64_t cover(int x0, int nX, int y0, int nY, GridRegion out[2]) {
    int64_t best = INT64_MAX;
    out[0] = out[1] = GridRegion{0, 0, 0, 0, false};
    if (nX <= 0 || nY <= 0) return 0;
    for (int swapped = 0; swapped < 2; ++swapped)
        for (int strip = 0; strip < 2; ++strip) {
            const int l0 = swapped ? y0 : x0, ln = swapped ? nY : nX;
            const int s0 = swapped ? x0 : y0, sn = swapped ? nX : nY;
            const int rest = ln % 64;
            if (strip && rest == 0) continue;
            const int main_n = strip ? ln - rest : ln;
            const int64_t cost = (int64_t)((main_n + 63) / 64) * quads_cost(sn) +
                                 (strip ? (int64_t)((sn + 63) / 64) * quads_cost(rest) : 0);
            if (cost >= best) continue;
            best = cost;
            out[0] = GridRegion{l0, main_n, s0, main_n ? sn : 0, swapped != 0};
            out[1] = strip ? GridRegion{s0, sn, l0 + main_n, rest, swapped == 0}
                           : GridRegion{0, 0, 0, 0, false};
        }
    return best;
}

// Jobs of `step` step positions.
static void count_jobs(GridPlan* p, int step) {
    p->step = step;
    p->jobs = p->oct_jobs + p->diag_jobs;
    for (int r = 0; r < 3; ++r) {
        const GridRegion& R = p->region[r];
        p->region_jobs[r] = (int64_t)((R.lane_n + 63) / 64) * ((R.step_n + step - 1) / step);
        p->jobs += p->region_jobs[r];
    }
}

bool grid_plan(int nx, int ny, int cx, int cy, double cell, int prec, GridGeom* g, GridPlan* p) {
    const bool f32 = prec == SWV_F32C;
    int64_t x0, nX, y0, nY;
    axis_offsets(nx, cx, &x0, &nX);
    axis_offsets(ny, cy, &y0, &nY);
    // offsets are used as ints; a centre that far away shares nothing anyway
    if (x0 + nX > (int64_t(1) << 30) || y0 + nY > (int64_t(1) << 30)) return false;
    *g = GridGeom{(int)x0, (int)nX, (int)y0, (int)nY, cell};
    *p = GridPlan{};
    const int Kx = (int)nX, Ky = (int)nY;
    // whole 64 x 64 blocks of the square in which (i, k) and (k, i) have one n
    int nb = x0 == y0 ? (Kx < Ky ? Kx : Ky) / 64 : 0;
    if (nb < 2 || f32) nb = 0;
    const int64_t b = nb;
    const int sq = 64 * nb;
    p->oct_jobs = 16 * b * (b - 1);
    p->diag_jobs = b * (64 / kStep);
    int64_t cost = p->oct_jobs * 33 * kOct + p->diag_jobs * quads_cost(kStep);
    // beside the square: x from sq on, then, over the square, y from sq on
    cost += cover(sq, Kx - sq, 0, Ky, p->region);
    if (sq > 0 && Ky > sq) {
        cost += b * quads_cost(Ky - sq);   // whole lane tiles along x
        p->region[2] = GridRegion{0, sq, sq, Ky - sq, false};
    }
    count_jobs(p, f32 ? kF32Step : kStep);
    // against 20 instructions per pixel of the general adjoint, whose idle lanes
    // are few: 256^2 about its centre 5,400 for quads and octets, 20,480 for pixels
    const int64_t pixel_waves = ((int64_t)nx * ny + 63) / 64;
    // FP32-compensated: about 78 issue slots of FP32 size per row and quad (20 of
    // each pixel's 26 in the adjoint)
    if (f32) return 78 * (cost / 25) <= 26 * pixel_waves;
    // the tables' 16 bytes a position, written and read, take the time of about four
    // more instructions each, which is what a thin image saves and more (1 x 300 pixels
    // of 100,000 rows: 159 us through tables, 77 by pixels)
    return cost + 4 * (nX + nY) <= 20 * pixel_waves;
}

// Rows per chunk: four rounds of workgroups (two per CU) rather than one, since
// the dies' clocks differ, while the partial sums stay within 256 MiB (8 chunks at
// least); 64 rows at least, so that filling the table stays small beside them, and
// fewer (8 at least) where that leaves less than four waves to a CU: they run at a
// row's latency (100 rows of 64 x 64 pixels, the whole call: 45 us in chunks of 64, 18.6
// in chunks of 8).
int64_t grid_chunk(const GridGeom& g, const GridPlan& p, int64_t rows, int n_cu) {
    const int64_t fill = 4 * (int64_t)n_cu * 2 * (kTabBlock / 64) / p.jobs;
    const int64_t cap = (int64_t(256) << 20) / (32 * (int64_t)g.Kx * g.Ky);
    const int64_t chunks = fill < cap ? (fill < 8 ? 8 : fill) : (cap < 8 ? 8 : cap);
    int64_t least = 64;
    while (least > 8 && p.jobs * ((rows + least - 1) / least) < 4 * (int64_t)n_cu) least /= 2;
    const int64_t chunk = (rows + chunks - 1) / chunks;
    return chunk < least ? least : (chunk < (int64_t(1) << 30) ? chunk : int64_t(1) << 30);
}

size_t grid_row_bytes(const GridGeom& g) {
    return sizeof(GridRow) + sizeof(Cell) * ((size_t)g.Kx + (size_t)g.Ky);
}

size_t grid_slab_bytes(const GridGeom& g, int64_t rows) {
    // kStep cells past the last row: a wave's scalar loads may run over the end
    return grid_row_bytes(g) * (size_t)rows + 2 * kStep * sizeof(Cell);
}

size_t grid_partial_bytes(const GridGeom& g, int64_t n_chunks) {
    return 32 * (size_t)g.Kx * (size_t)g.Ky * (size_t)n_chunks;
}

hipError_t launch_grid_slab(hipStream_t s, const GridGeom& g, const GridPlan& p, int64_t rows,
                            int64_t chunk, const double* u, const double* v, const double* w,
                            const void* y, int sign, bool resume, void* slab, double* partial) {
    if (rows <= 0) return hipSuccess;
    GridRow* rec = (GridRow*)slab;
    Cell* ex = (Cell*)(rec + rows);
    Cell* ey = ex + (size_t)g.Kx * (size_t)rows + kStep;
    const int64_t items = rows * ((int64_t)g.Kx + g.Ky);
    const int64_t nb = (items + 255) / 256;
    k_grid_prep<<<dim3((unsigned)(nb < 65536 ? nb : 65536)), dim3(256), 0, s>>>(
        u, v, w, (const double2*)y, rows, g, sign > 0 ? -1.0 : 1.0, rec, ex, ey);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t jobs = (rows + chunk - 1) / chunk * p.jobs;
    const int64_t per = kTabBlock / 64, run = ((jobs + per - 1) / per + 7) / 8;
    if (8 * run > kMaxLaunchThreads / kTabBlock) return hipErrorInvalidConfiguration;
    const GridData data{rec, ex, ey, partial, resume};
    const dim3 grid((unsigned)(8 * run)), blk(kTabBlock);
    if (y)
        k_grid_sums<false><<<grid, blk, 0, s>>>(g, p, rows, chunk, jobs, run, data);
    else
        k_grid_sums<true><<<grid, blk, 0, s>>>(g, p, rows, chunk, jobs, run, data);
    return hipGetLastError();
}

hipError_t launch_image_f32c(hipStream_t s, const GridGeom& g, const GridPlan& plan, int64_t n_vis,
                             int64_t chunk, int n_cu, const double* u, const double* v,
                             const double* w, const void* y, int sign, double* partial) {
    // one quad a lane where two leave less than eight waves to a CU (1,000 rows of 256 x
    // 256 pixels, the whole call: 41 and 52 us)
    GridPlan p = plan;
    if (p.jobs * ((n_vis + chunk - 1) / chunk) < 8 * (int64_t)n_cu) count_jobs(&p, 1);
    const int64_t jobs = (n_vis + chunk - 1) / chunk * p.jobs;
    const int64_t per = kF32Block / 64, run = ((jobs + per - 1) / per + 7) / 8;
    if (8 * run > kMaxLaunchThreads / kF32Block) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)(8 * run)), blk(kF32Block);
    const float fsg = (float)sign;
    if (y)
        k_image_f32c<false><<<grid, blk, 0, s>>>(g, p, u, v, w, (const double2*)y, n_vis, chunk,
                                                 jobs, run, fsg, partial);
    else
        k_image_f32c<true><<<grid, blk, 0, s>>>(g, p, u, v, w, nullptr, n_vis, chunk, jobs, run,
                                                fsg, partial);
    return hipGetLastError();
}

hipError_t launch_grid_finish(hipStream_t s, const GridGeom& g, int prec, const double* partial,
                              int64_t n_chunks, int nx, int ny, int cx, int cy, int64_t n_vis,
                              double* img) {
    const int64_t cols = 4 * (int64_t)g.Kx * g.Ky;
    const int per = kFinCols * 4, block = per * kFinQ;
    launch_slabs((cols + per - 1) / per, block, [&](int64_t b0, unsigned nb) {
        if (prec == SWV_F32C)
            k_grid_finish<true><<<dim3(nb), dim3(block), 0, s>>>(
                g, partial, n_chunks, b0, nx, ny, cx, cy, (double)n_vis, img);
        else
            k_grid_finish<false><<<dim3(nb), dim3(block), 0, s>>>(
                g, partial, n_chunks, b0, nx, ny, cx, cy, (double)n_vis, img);
    });
    return hipGetLastError();
}

}  // namespace swv
