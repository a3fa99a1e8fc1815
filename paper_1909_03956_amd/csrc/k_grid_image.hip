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
// adjoint takes 20 (table phasor) and throws its imaginary half away.  Bound by
// FP64 issue: 176,904 rows x 256^2 pixels 19.6 -> 2.95 ms, the same of a 511^2
// beam (y = 1, 21 instructions) 60 -> 10.4 ms, about 70 % of the issue rate at
// 2.4 GHz.  With every table read from one row instead: 2.81 and 9.6 ms, so the
// loads are nearly hidden.
//
// Accuracy: the phases u l, v m are reduced with their products' rounding
// errors, w (n - 1) enters the cell search and the rest by FMAs, so no phase is
// rounded at its own magnitude; each phasor is good to a few 2^-53.
//
// Layout.  A prep kernel writes, for a slab of rows, {w, y} records and the
// tables E_x, E_y (16 (Kx + Ky) + 32 bytes a row; slabs bound the workspace).
// A wave takes 64 neighbouring |k| of one axis (the lane axis, E by coalesced
// vector loads) and up to four of the other (E by scalar loads, an SGPR operand
// of every lane's products).  Kx is rarely a multiple of 64 (129 for a 256-pixel
// side), so what is left over beyond whole waves of one axis is covered by a
// strip with the axes exchanged.
#include "chunking.h"
#include "device_math.h"
#include "launch.h"
#include "phasor_table.h"

namespace swv {

namespace {

constexpr int kStep = 4;   // scalar-axis positions per wave

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

// acc[i] += (P, lane-sine products Q and R, step-sine product S) of row
// (w, z = y): UNIT for y = 1.
template <int G, bool UNIT, bool WIDE>
__device__ __forceinline__ void add_row(CellPtr T, const CellCoefs& K, double w, double yr, double yi, Cell a,
                                        ScalarCells b, const double (&nm1)[G],
                                        double (&acc)[G][4]) {
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
        const double zr = fma(e[i].x, tr, -(e[i].y * ti));
        const double zi = fma(e[i].x, ti, e[i].y * tr);
        const double cb = b[i].x, sb = b[i].y;
        acc[i][0] = fma(zr * a.x, cb, acc[i][0]);
        acc[i][1] = fma(zr * a.y, sb, acc[i][1]);
        acc[i][2] = fma(zi * a.y, cb, acc[i][2]);
        acc[i][3] = fma(zi * a.x, sb, acc[i][3]);
    }
}

template <int G, bool UNIT, bool WIDE>
__device__ __forceinline__ void add_rows(CellPtr T, const CellCoefs& K, RowPtr R, int nrow,
                                         const Cell* __restrict__ A, int KA, ScalarCells B, int KB,
                                         const double (&nm1)[G], double (&acc)[G][4]) {
    Cell next = A[0];
#pragma unroll 1
    for (int j = 0; j < nrow; ++j) {
        const Cell a = next;
        next = A[(int64_t)(j + 1 < nrow ? j + 1 : j) * KA];   // ahead of this row's arithmetic
        add_row<G, UNIT, WIDE>(T, K, R[j].w, R[j].yr, R[j].yi, a, B + (int64_t)j * KB, nm1, acc);
    }
}

// One wave's quads (lane position `lane`, step positions step0 .. step0 + G) over
// the rows of a chunk.
template <int G, bool UNIT>
__device__ __forceinline__ void grid_wave(CellPtr T, const GridGeom& g, bool swapped, int lane,
                                          int lane_end, int step, int step_end, int64_t j0,
                                          int nrow, const GridRow* rec, const Cell* ex,
                                          const Cell* ey, bool wide, bool resume, int64_t quad_base,
                                          double* partial) {
    const int la = lane < lane_end ? lane : lane_end - 1;   // idle lanes repeat the last
    const int KA = swapped ? g.Ky : g.Kx, KB = swapped ? g.Kx : g.Ky;
    const Cell* __restrict__ A = (swapped ? ey : ex) + j0 * KA + la;
    ScalarCells B = uniform_ptr((swapped ? ex : ey) + j0 * KB + step);
    RowPtr R = uniform_ptr(rec + j0);
    double nm1[G], acc[G][4];
    int64_t quad[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int st = step + i < step_end ? step + i : step_end - 1;
        const int kx = swapped ? st : la, ky = swapped ? la : st;
        nm1[i] = g.nm1(kx, ky);
        quad[i] = quad_base + (int64_t)ky * g.Kx + kx;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            acc[i][t] = resume ? partial[4 * quad[i] + (swapped && t >= 2 ? 5 - t : t)] : 0.0;
    }
    const CellCoefs K = cell_coefs();
    if (__builtin_expect(wide, 0))
        add_rows<G, UNIT, true>(T, K, R, nrow, A, KA, B, KB, nm1, acc);
    else
        add_rows<G, UNIT, false>(T, K, R, nrow, A, KA, B, KB, nm1, acc);
#pragma unroll
    for (int i = 0; i < G; ++i) {
        if (lane < lane_end && step + i < step_end) {
            // exchanged axes: R and S change places
            double2* o = (double2*)(partial + 4 * quad[i]);
            o[0] = make_double2(acc[i][0], acc[i][1]);
            o[1] = swapped ? make_double2(acc[i][3], acc[i][2]) : make_double2(acc[i][2], acc[i][3]);
        }
    }
}

}  // namespace

// Block (chunk, tile): the tile's waves take consecutive jobs, first those of
// the main region, then the strip's.
template <bool UNIT>
__global__ __launch_bounds__(kTabBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_grid_sums(
    GridGeom g, GridPlan p, int64_t n_rows, int64_t chunk, int64_t n_chunks, int64_t bid0,
    const GridRow* __restrict__ rec, const Cell* __restrict__ ex, const Cell* __restrict__ ey,
    bool resume, double* __restrict__ partial) {
    __shared__ Cell T[kTabCells];
    int64_t chunk_id, tile;
    chunk_tile(bid0 + blockIdx.x, p.tiles, chunk_id, tile);
    if (chunk_id >= n_chunks) return;   // padding of the last XCD group (whole block)
    fill_cells(T);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t job = tile * (kTabBlock / 64) + wave;
    const bool strip = job >= p.jobs[0];
    if (strip) job -= p.jobs[0];
    if (job >= p.jobs[strip]) return;
    // (region, exchanged) of a job; lane tiles run fastest, so neighbouring waves
    // share their scalar-axis positions
    const int region = __builtin_amdgcn_readfirstlane(strip ? 1 : 0);
    const int lane0 = p.lane0[region], lane_end = lane0 + p.lane_n[region];
    const int step0 = p.step0[region], step_end = step0 + p.step_n[region];
    const bool swapped = p.swapped != (region == 1);
    const int lt = (p.lane_n[region] + 63) / 64;
    const int la = lane0 + (int)(job % lt) * 64 + lane;
    const int step = __builtin_amdgcn_readfirstlane(step0 + (int)(job / lt) * kStep);
    const int left = step_end - step;
    const int64_t j0 = chunk_id * chunk;
    const int nrow = __builtin_amdgcn_readfirstlane(
        (int)(j0 + chunk < n_rows ? chunk : n_rows - j0));
    const int64_t base = chunk_id * (int64_t)g.Kx * g.Ky;
    const CellPtr TP = (CellPtr)T;
    // a row that needs the WIDE form puts the whole chunk through it
    bool any = false;
    for (int j = lane; j < nrow; j += 64) any = any || rec[j0 + j].wide != 0;
    const bool wide = __any(any);
    if (left > 2)
        grid_wave<4, UNIT>(TP, g, swapped, la, lane_end, step, step_end, j0, nrow, rec, ex, ey,
                           wide, resume, base, partial);
    else if (left == 2)
        grid_wave<2, UNIT>(TP, g, swapped, la, lane_end, step, step_end, j0, nrow, rec, ex, ey,
                           wide, resume, base, partial);
    else
        grid_wave<1, UNIT>(TP, g, swapped, la, lane_end, step, step_end, j0, nrow, rec, ex, ey,
                           wide, resume, base, partial);
}

// Adds the chunks of each quad (16 threads take every 16th chunk in order, their
// sums meet in a fixed tree) and writes its pixels: 0 off the unit disk.
constexpr int kFinCols = 16, kFinQ = 16;

__global__ __launch_bounds__(kFinCols * 4 * kFinQ) void k_grid_finish(
    GridGeom g, const double* __restrict__ partial, int64_t n_chunks, int nx, int ny, int cx, int cy,
    double n_vis, double* __restrict__ img) {
    __shared__ double red[kFinQ][kFinCols * 4];
    const int64_t quads = (int64_t)g.Kx * g.Ky;
    const int tx = threadIdx.x % (kFinCols * 4), r = threadIdx.x / (kFinCols * 4);
    const int64_t at = (int64_t)blockIdx.x * (kFinCols * 4) + tx;   // 4 quad + component
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
    const double v = (q4[0] - (sl * sm) * q4[1]) - (sl * q4[2] + sm * q4[3]);
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

// Waves of a cover: the whole lane tiles, and the rest either as one more,
// partly idle lane tile or as a strip with the axes exchanged.
static int64_t cover(int64_t lane_n, int64_t step_n, bool strip) {
    if (!strip) return (lane_n + 63) / 64 * step_n;
    return lane_n / 64 * step_n + lane_n % 64 * ((step_n + 63) / 64);
}

bool grid_plan(int nx, int ny, int cx, int cy, double cell, GridGeom* g, GridPlan* p) {
    int64_t x0, nX, y0, nY;
    axis_offsets(nx, cx, &x0, &nX);
    axis_offsets(ny, cy, &y0, &nY);
    // offsets are used as ints; a centre that far away shares nothing anyway
    if (x0 + nX > (int64_t(1) << 30) || y0 + nY > (int64_t(1) << 30)) return false;
    *g = GridGeom{(int)x0, (int)nX, (int)y0, (int)nY, cell};
    int64_t best = INT64_MAX;
    for (int swapped = 0; swapped < 2; ++swapped)
        for (int strip = 0; strip < 2; ++strip) {
            const int64_t ln = swapped ? nY : nX, sn = swapped ? nX : nY;
            if (strip && (ln % 64 == 0)) continue;
            const int64_t waves = cover(ln, sn, strip != 0);
            if (waves >= best) continue;
            best = waves;
            *p = GridPlan{};
            p->swapped = swapped != 0;
            const int main_n = (int)(strip ? ln / 64 * 64 : ln);
            p->lane_n[0] = main_n;
            p->step_n[0] = main_n ? (int)sn : 0;
            if (strip) {   // axes exchanged: lanes along the other axis
                p->lane_n[1] = (int)sn;
                p->step0[1] = main_n;
                p->step_n[1] = (int)(ln - main_n);
            }
        }
    for (int r = 0; r < 2; ++r)
        p->jobs[r] = (int64_t)((p->lane_n[r] + 63) / 64) * ((p->step_n[r] + kStep - 1) / kStep);
    const int per_block = kTabBlock / 64;
    p->tiles = (p->jobs[0] + p->jobs[1] + per_block - 1) / per_block;
    // 25 instructions per quad and row against 20 per pixel of the general
    // adjoint (its idle lanes are few): 256^2 about its centre 264 waves of quads
    // against 1,024 of pixels
    const int64_t pixel_waves = ((int64_t)nx * ny + 63) / 64;
    return 25 * best <= 20 * pixel_waves;
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

int grid_blocks_per_cu() { return 2; }

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
    const int64_t n_chunks = (rows + chunk - 1) / chunk;
    launch_slabs(xcd_padded(n_chunks) * p.tiles, [&](int64_t b0, unsigned b) {
        if (y)
            k_grid_sums<false><<<dim3(b), dim3(kTabBlock), 0, s>>>(g, p, rows, chunk, n_chunks, b0,
                                                                   rec, ex, ey, resume, partial);
        else
            k_grid_sums<true><<<dim3(b), dim3(kTabBlock), 0, s>>>(g, p, rows, chunk, n_chunks, b0,
                                                                  rec, ex, ey, resume, partial);
    });
    return hipGetLastError();
}

hipError_t launch_grid_finish(hipStream_t s, const GridGeom& g, const double* partial,
                              int64_t n_chunks, int nx, int ny, int cx, int cy, int64_t n_vis,
                              double* img) {
    const int64_t cols = 4 * (int64_t)g.Kx * g.Ky;
    const int per = kFinCols * 4;
    k_grid_finish<<<dim3((unsigned)((cols + per - 1) / per)), dim3(per * kFinQ), 0, s>>>(
        g, partial, n_chunks, nx, ny, cx, cy, (double)n_vis, img);
    return hipGetLastError();
}

}  // namespace swv
