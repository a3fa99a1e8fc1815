// Major-cycle kernels around the prediction: the subtract step with chi^2
// (section 2.2), the exact adjoint of the direct sum (the residual image on
// sphere pixels), and the chi^2 gradients of the direct sum.
//
// Adjoint and gradients swap the roles of the direct kernel: lanes own the
// outputs (pixels or components) and every lane of the wave walks the same
// visibility rows, read with scalar loads.  The visibility axis is split into
// fixed chunks whose partial sums a second kernel adds in a fixed order --
// deterministic and free of atomics.
#include <algorithm>
#include <type_traits>

#include "chunking.h"
#include "device_math.h"
#include "launch.h"
#include "phasor_table.h"

namespace swv {

// ---------------------------------------------------------------- adjoint --
// img[p] = sum_j conj(e_jp) y_j, e = exp(s 2 pi i phi).
//
// FP64: one wave per (chunk of rows, column of up to four groups of 64 pixels).
// With the pixels' directions times -s, conj(e) = exp(2 pi i phi) = node x rest,
// and y is turned by the rest, then by the node straight into the sums: 20 FP64
// instructions per row and pixel (phase 3, cell 4, rest 5, 4 + 4), against 29
// with the polynomial phasor; bound by their issue.  8,355,840 rows x 955
// pixels: 7.48 -> 5.14 ms (83 % of the issue rate at 2.4 GHz; the clock under this
// load is about 1.9).
//
// Workgroups of 512 threads (two share a CU, a 64 KB table each).  Up to 32 groups
// make 1, 2, 4 or 8 columns, and a workgroup takes a chunk: its waves the columns
// and, by parts, the chunk's rows; the parts' sums meet in LDS where the table
// was, so there is one set of partial sums per workgroup and four rounds of them stay
// small: 955 pixels 5.58 -> 5.14 ms against a chunk per wave and two rounds, 40
// pixels x 5,000,000 rows 0.322 -> 0.291.  More columns are numbered chunk-major and dealt to the
// waves in order.  Workgroups go to the XCDs in runs (their ids go round-robin), so
// a chunk's rows come into one L2 and no workgroup is partly idle but the last.
constexpr int kAdjWaves = kTabBlock / 64;
// rows per step: 1, 2 and 4 take 0.708, 0.485 and 0.394 ms on 5,000,000 rows x 40
// pixels, where the rows' loads show (and 5.57, 5.53 and 5.52 ms on 955 pixels), with a
// chunk per wave
constexpr int kAdjRows = 4;
constexpr int64_t kAdjMinRows = 32;

// How n outputs go to waves: `groups` of 64 in `cols` columns; `parts` waves of a
// workgroup share a column's rows (1: columns past eight, dealt wave by wave).
struct Columns {
    int64_t groups, cols;
    int parts;
};

static Columns columns_of(int64_t n, int per_lane) {
    Columns c;
    c.groups = (n + 63) / 64;
    c.cols = (c.groups + per_lane - 1) / per_lane;
    c.parts = 1;
    if (c.cols <= kAdjWaves) {
        int64_t p = 1;
        while (p < c.cols) p *= 2;
        c.cols = p;
        c.parts = kAdjWaves / (int)p;
    }
    return c;
}

// What a wave does: rows j0 .. j0 + nrow of chunk `chunk`, the G groups of 64
// outputs from group g0 (the groups spread evenly over the columns).  active is
// false past the last job.
struct WaveJob {
    int64_t chunk, j0, g0;
    int nrow, G, part, slot;   // slot: of the wave's sums in LDS (part > 0)
    bool active;
};
__device__ __forceinline__ WaveJob wave_job(int64_t n_vis, int64_t chunk, const Columns& C,
                                            int64_t n_chunks, int64_t run) {
    const int64_t bid = blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t blk = (bid & 7) * run + (bid >> 3);
    WaveJob w;
    int64_t c, end;
    if (C.parts > 1 || C.cols == kAdjWaves) {
        c = wave % (int)C.cols;
        w.part = wave / (int)C.cols;
        w.chunk = blk;
        const int64_t sub = (chunk + C.parts - 1) / C.parts;
        w.j0 = blk * chunk + w.part * sub;
        end = w.part + 1 < C.parts ? w.j0 + sub : (blk + 1) * chunk;
        end = end < (blk + 1) * chunk ? end : (blk + 1) * chunk;
        w.slot = (w.part - 1) * (int)C.cols + (int)c;
    } else {
        const int64_t job = blk * kAdjWaves + wave;
        w.chunk = job / C.cols;
        c = job - w.chunk * C.cols;
        w.part = w.slot = 0;
        w.j0 = w.chunk * chunk;
        end = w.j0 + chunk;
    }
    w.active = w.chunk < n_chunks;
    end = end < n_vis ? end : n_vis;
    if (!w.active) w.chunk = w.j0 = c = end = 0;
    w.nrow = __builtin_amdgcn_readfirstlane(end > w.j0 ? (int)(end - w.j0) : 0);
    w.g0 = c * C.groups / C.cols;
    w.G = __builtin_amdgcn_readfirstlane((int)((c + 1) * C.groups / C.cols - w.g0));
    return w;
}

// Adds the sums of a column's parts in order: x[t][i] for the group i < G.  All
// waves of the workgroup call it (it takes the table's place); true in the waves
// that hold the result.
template <int N>
__device__ __forceinline__ bool join_parts(Cell* T, const WaveJob& job, const Columns& C,
                                           double (&x)[N][4]) {
    static_assert(N % 2 == 0 && (kAdjWaves - 1) * 4 * 64 * (N / 2) <= kTabCells, "fits the table");
    if (C.parts == 1) return job.active;
    const int lane = threadIdx.x & 63;
    const auto at = [&](int slot, int i, int h) {
        return ((slot * 4 + i) * (N / 2) + h) * 64 + lane;
    };
    __syncthreads();   // every wave is done with the table
    if (job.part > 0)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < job.G)
#pragma unroll
                for (int h = 0; h < N / 2; ++h)
                    T[at(job.slot, i, h)] = Cell{x[2 * h][i], x[2 * h + 1][i]};
    __syncthreads();
    if (job.part > 0) return false;
    for (int k = 1; k < C.parts; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < job.G)
#pragma unroll
                for (int h = 0; h < N / 2; ++h) {
                    const Cell p = T[at(job.slot + k * (int)C.cols, i, h)];
                    x[2 * h][i] += p.x;
                    x[2 * h + 1][i] += p.y;
                }
    return job.active;
}

// Whether a row of the wave's chunk has phases that need the WIDE form (or are
// not finite): the whole chunk then goes through it.
__device__ __forceinline__ bool chunk_is_wide(const WaveJob& job, const double* __restrict__ u,
                                              const double* __restrict__ v,
                                              const double* __restrict__ w) {
    bool big = false;
    for (int j = threadIdx.x & 63; j < job.nrow; j += 64)
        big = big || !cells_reach(u[job.j0 + j], v[job.j0 + j], w[job.j0 + j]);
    return __any(big);
}

template <int G, bool WIDE>
__device__ __forceinline__ void adjoint_rows(
    CellPtr T, const double* u, const double* v, const double* w, const double2* y, int nrow,
    const double (&L)[G], const double (&M)[G], const double (&N)[G], double (&ar)[G],
    double (&ai)[G]) {
    const auto* U = uniform_ptr(u);
    const auto* V = uniform_ptr(v);
    const auto* W = uniform_ptr(w);
    const auto* Y = uniform_ptr(y);
    const CellCoefs K = cell_coefs();
    // R rows per step: their scalar loads go out together
    const auto step = [&](auto rows, int j) {
        constexpr int R = decltype(rows)::value;
        double uj[R], vj[R], wj[R], yr[R], yi[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uj[r] = U[j + r];
            vj[r] = V[j + r];
            wj[r] = W[j + r];
            yr[r] = Y[j + r].x;
            yi[r] = Y[j + r].y;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            Cell e[G];
            double d[G];
#pragma unroll
            for (int i = 0; i < G; ++i)
                e[i] = find_cell<WIDE>(T, fma(uj[r], L[i], fma(vj[r], M[i], wj[r] * N[i])), d[i],
                                       K.magic);
#pragma unroll
            for (int i = 0; i < G; ++i) {
                double cr, sr;
                cell_rest(K, d[i], cr, sr);
                const double tr = fma(cr, yr[r], -(sr * yi[r]));
                const double ti = fma(cr, yi[r], sr * yr[r]);
                ar[i] = fma(e[i].x, tr, ar[i]);
                ai[i] = fma(e[i].x, ti, ai[i]);
                ar[i] = fma(-e[i].y, ti, ar[i]);
                ai[i] = fma(e[i].y, tr, ai[i]);
            }
        }
    };
    int j = 0;
#pragma unroll 1
    for (; j + kAdjRows <= nrow; j += kAdjRows) step(std::integral_constant<int, kAdjRows>(), j);
#pragma unroll 1
    for (; j < nrow; ++j) step(std::integral_constant<int, 1>(), j);
}

// x[0], x[1]: the sums' real and imaginary parts.
template <int G>
__device__ __forceinline__ void adjoint_wave(
    CellPtr T, const double* __restrict__ u, const double* __restrict__ v,
    const double* __restrict__ w, const double2* __restrict__ y, int nrow, bool wide,
    const double* __restrict__ pl, const double* __restrict__ pm, const double* __restrict__ pn,
    int64_t q0, int64_t n_pix, double sgn, double (&x)[2][4]) {
    double L[G], M[G], N[G], ar[G], ai[G];
    bool far = false;
#pragma unroll
    for (int i = 0; i < G; ++i) {
        int64_t p = q0 + (int64_t)i * 64;
        p = p < n_pix ? p : n_pix - 1;
        L[i] = -sgn * pl[p];
        M[i] = -sgn * pm[p];
        N[i] = -sgn * pn[p];
        far = far || !(fabs(L[i]) <= 2.0 && fabs(M[i]) <= 2.0 && fabs(N[i]) <= 2.0);
        ar[i] = ai[i] = 0.0;
    }
    if (__builtin_expect(wide || __any(far), 0))
        adjoint_rows<G, true>(T, u, v, w, y, nrow, L, M, N, ar, ai);
    else
        adjoint_rows<G, false>(T, u, v, w, y, nrow, L, M, N, ar, ai);
#pragma unroll
    for (int i = 0; i < G; ++i) {
        x[0][i] = ar[i];
        x[1][i] = ai[i];
    }
}

__global__ __launch_bounds__(kTabBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_adjoint_cell(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    const double2* __restrict__ y, int64_t n_vis, int64_t chunk, const double* __restrict__ pl,
    const double* __restrict__ pm, const double* __restrict__ pn, int64_t n_pix, double sgn,
    Columns C, int64_t n_chunks, int64_t run, double2* __restrict__ partial) {
    __shared__ Cell T[kTabCells];
    const WaveJob job = wave_job(n_vis, chunk, C, n_chunks, run);
    const bool wide = chunk_is_wide(job, u, v, w);
    fill_cells(T);
    const int64_t j0 = job.j0, q0 = job.g0 * 64 + (threadIdx.x & 63);
    const CellPtr TP = (CellPtr)T;
    double x[2][4] = {};
#define SWV_WAVE(N)                                                                          \
    adjoint_wave<N>(TP, u + j0, v + j0, w + j0, y + j0, job.nrow, wide, pl, pm, pn, q0, n_pix, \
                    sgn, x)
    switch (job.nrow > 0 ? job.G : 0) {
        case 0: break;
        case 1: SWV_WAVE(1); break;
        case 2: SWV_WAVE(2); break;
        case 3: SWV_WAVE(3); break;
        default: SWV_WAVE(4); break;
    }
#undef SWV_WAVE
    if (!join_parts<2>(T, job, C, x)) return;
    double2* part = partial + job.chunk * n_pix;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t p = q0 + (int64_t)i * 64;
        if (i < job.G && p < n_pix) part[p] = make_double2(x[0][i], x[1][i]);
    }
}

// FP32-compensated: FP64 phase reduced exactly; FP32 phasor, products and Kahan
// sums.  One lane's G pixels q0, q0 + 64, ... over the rows of chunk chunk_id.
// With e = c + i s S: conj(e) y = (c yr + s S yi) + i (c yi - s S yr).
template <int G>
__device__ __forceinline__ void adjoint_lane_f32c(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    const double2* __restrict__ y, int64_t n_vis, int64_t chunk, const double* __restrict__ pl,
    const double* __restrict__ pm, const double* __restrict__ pn, int64_t n_pix, double sgn,
    int64_t chunk_id, int64_t q0, double2* __restrict__ partial) {
    double L[G], M[G], N[G];
    float sr[G], cr[G], si[G], ci[G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        int64_t p = q0 + (int64_t)i * 64;
        p = p < n_pix ? p : n_pix - 1;
        L[i] = pl[p];
        M[i] = pm[p];
        N[i] = pn[p];
        sr[i] = cr[i] = si[i] = ci[i] = 0.0f;
    }
    const int64_t j0 = chunk_id * chunk;
    const int64_t j1 = j0 + chunk < n_vis ? j0 + chunk : n_vis;
    // wave-uniform trip count, kept in scalar registers
    const int nrow = __builtin_amdgcn_readfirstlane((int)(j1 - j0));
    const auto* U = uniform_ptr(u + j0);
    const auto* V = uniform_ptr(v + j0);
    const auto* W = uniform_ptr(w + j0);
    const auto* Y = uniform_ptr(y + j0);
    // rows in pairs: the pair's four products and the running compensation
    // meet in one chain of FMAs, then one Kahan step, so a row costs half a
    // step (the chain's roundings stay within a few 2^-24 of the pair's
    // terms); an odd last row enters alone
    // sgn is +-1, so fsg * (float)y is (float)(sgn * y) bit for bit
    const float fsg = (float)sgn;
    const auto cis = [&](double uj, double vj, double wj, int i, float& c, float& s) {
        cis2pi_f32((float)fract_phase(uj, vj, wj, L[i], M[i], N[i]), c, s);
    };
    const int npair = nrow & ~1;
#pragma unroll 2
    for (int j = 0; j < npair; j += 2) {
        const double u0 = U[j], v0 = V[j], w0 = W[j], yr0 = Y[j].x, yi0 = Y[j].y;
        const double u1 = U[j + 1], v1 = V[j + 1], w1 = W[j + 1];
        const double yr1 = Y[j + 1].x, yi1 = Y[j + 1].y;
        const float fyr0 = (float)yr0, fyi0 = (float)yi0;
        const float fsyr0 = fsg * fyr0, fsyi0 = fsg * fyi0;
        const float fyr1 = (float)yr1, fyi1 = (float)yi1;
        const float fsyr1 = fsg * fyr1, fsyi1 = fsg * fyi1;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            float c0, s0, c1, s1;
            cis(u0, v0, w0, i, c0, s0);
            cis(u1, v1, w1, i, c1, s1);
            kahan_step(fmaf(c0, fyr0, fmaf(s0, fsyi0, fmaf(c1, fyr1, fmaf(s1, fsyi1, -cr[i])))),
                       sr[i], cr[i]);
            kahan_step(fmaf(c0, fyi0, fmaf(-s0, fsyr0, fmaf(c1, fyi1, fmaf(-s1, fsyr1, -ci[i])))),
                       si[i], ci[i]);
        }
    }
    if (npair < nrow) {
        const int j = npair;
        const double yr = Y[j].x, yi = Y[j].y;
        const float fyr = (float)yr, fyi = (float)yi;
        const float fsyr = fsg * fyr, fsyi = fsg * fyi;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            float c, s;
            cis(U[j], V[j], W[j], i, c, s);
            kahan_step(fmaf(c, fyr, fmaf(s, fsyi, -cr[i])), sr[i], cr[i]);
            kahan_step(fmaf(c, fyi, fmaf(-s, fsyr, -ci[i])), si[i], ci[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < G; ++i) {
        const int64_t p = q0 + (int64_t)i * 64;
        if (p < n_pix)
            partial[chunk_id * n_pix + p] =
                make_double2((double)sr[i] - (double)cr[i], (double)si[i] - (double)ci[i]);
    }
}

// Each wave of a tile owns PPL consecutive groups of 64 pixels (lane l of the
// wave takes pixel l of each group), so the pixels past the last one gather
// in whole groups at the end of the last tile, which are not computed (the
// 955-pixel image of the major cycle in one 1,024-pixel tile: 64 of its 69
// idle slots).  A pixel's sum is the same whichever lane takes it.
template <int PPL, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_adjoint_f32c(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    const double2* __restrict__ y, int64_t n_vis, int64_t chunk, const double* __restrict__ pl,
    const double* __restrict__ pm, const double* __restrict__ pn, int64_t n_pix, double sgn,
    int64_t n_chunks, int64_t tiles, int64_t bid0, double2* __restrict__ partial) {
    int64_t chunk_id, tile;
    chunk_tile(bid0 + blockIdx.x, tiles, chunk_id, tile);
    if (chunk_id >= n_chunks) return;   // padding of the last XCD group
    static_assert(BLOCK % 64 == 0, "whole waves");
    const int wave = (int)(threadIdx.x / 64), lane = (int)(threadIdx.x % 64);
    const int64_t g0 = tile * (BLOCK * PPL) + (int64_t)wave * (64 * PPL);
    const int64_t left = n_pix - g0;   // the same for every lane of the wave
    const int groups = __builtin_amdgcn_readfirstlane(
        left <= 0 ? 0 : (left >= 64 * PPL ? PPL : (int)((left + 63) / 64)));
    const int64_t q0 = g0 + lane;
    if (groups >= PPL) {
        adjoint_lane_f32c<PPL>(u, v, w, y, n_vis, chunk, pl, pm, pn, n_pix, sgn, chunk_id, q0,
                                partial);
    } else if constexpr (PPL >= 2) {
        if (groups == 1)
            adjoint_lane_f32c<1>(u, v, w, y, n_vis, chunk, pl, pm, pn, n_pix, sgn, chunk_id, q0,
                                  partial);
        if constexpr (PPL >= 4) {
            if (groups == 2)
                adjoint_lane_f32c<2>(u, v, w, y, n_vis, chunk, pl, pm, pn, n_pix, sgn, chunk_id,
                                      q0, partial);
            if (groups == 3)
                adjoint_lane_f32c<3>(u, v, w, y, n_vis, chunk, pl, pm, pn, n_pix, sgn, chunk_id,
                                      q0, partial);
        }
    }
}

// out[p] = sum over chunks c of partial[c][p].
// Chunk reductions: a block owns COLS consecutive outputs (coalesced along x); its
// Q rows of threads each add the chunks q, q + Q, ... in order, kAhead loads in
// flight, and the Q subtotals are then added by a fixed binary tree in LDS.  The
// order depends only on the counts of chunks and outputs, so results are run-to-run
// identical.  Few outputs are bound by the latency of a thread's chain and by the few
// blocks: 8 columns and 128 rows (955 outputs x 512 chunks: 3.0 us, 5.6 with 64 and
// 16).  Many are bound by their bytes, and by the blocks themselves where the chunks
// are few: 64 columns (10,000 x 152: 3.9 us, 5.1 with 16, 6.4 with 8), and 256 and 4
// rows for up to 24 chunks (1,000,000 x 2: 11 us, 36 with 64, 153 with 16).
constexpr int kSumBlock = 1024;
constexpr int64_t kSumNarrow = 4096;   // outputs below which a block takes 8
constexpr int64_t kSumFew = 24;        // chunks up to which it takes 256
constexpr int kAhead = 8;

template <int COLS>
__global__ __launch_bounds__(kSumBlock) void k_sum_chunks_c128(
    const double2* __restrict__ partial, int64_t n_chunks, int64_t n, int64_t bid0,
    double2* __restrict__ out) {
    constexpr int Q = kSumBlock / COLS;
    __shared__ double red_r[Q][COLS], red_i[Q][COLS];
    const int tx = threadIdx.x % COLS, q = threadIdx.x / COLS;
    const int64_t p = (bid0 + blockIdx.x) * COLS + tx;
    double re = 0.0, im = 0.0;
    if (p < n) {
        int64_t c = q;
        for (; c + (kAhead - 1) * Q < n_chunks; c += kAhead * Q) {
            double2 x[kAhead];
#pragma unroll
            for (int t = 0; t < kAhead; ++t) x[t] = partial[(c + t * Q) * n + p];
#pragma unroll
            for (int t = 0; t < kAhead; ++t) {
                re += x[t].x;
                im += x[t].y;
            }
        }
        for (; c < n_chunks; c += Q) {
            const double2 x = partial[c * n + p];
            re += x.x;
            im += x.y;
        }
    }
    red_r[q][tx] = re;
    red_i[q][tx] = im;
    __syncthreads();
    for (int h = Q / 2; h > 0; h >>= 1) {
        if (q < h) {
            red_r[q][tx] += red_r[q + h][tx];
            red_i[q][tx] += red_i[q + h][tx];
        }
        __syncthreads();
    }
    if (q == 0 && p < n) out[p] = make_double2(red_r[0][tx], red_i[0][tx]);
}

template <int PPL, int BLOCK>
static void run_adjoint_f32c(hipStream_t s, int64_t tiles, int64_t chunk, int64_t n_vis,
                             const double* u, const double* v, const double* w, const void* y,
                             int64_t n_pix, const double* l, const double* m, const double* nm1,
                             int sign, void* partial) {
    const int64_t n_chunks = (n_vis + chunk - 1) / chunk;
    launch_slabs(xcd_padded(n_chunks) * tiles, BLOCK, [&](int64_t b0, unsigned nb) {
        k_adjoint_f32c<PPL, BLOCK><<<dim3(nb), dim3(BLOCK), 0, s>>>(
            u, v, w, (const double2*)y, n_vis, chunk, l, m, nm1, n_pix, (double)sign, n_chunks,
            tiles, b0, (double2*)partial);
    });
}

// Blocks of one kernel shape that fit on a compute unit at once (registers,
// LDS, waves), from the runtime's occupancy calculator; cached per shape.
template <class K>
static int resident_blocks(K kernel, int block) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, block, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return nb > 0 ? nb : 1;
}

template <int PPL, int BLOCK>
static int adjoint_f32c_occ() {
    static const int v = resident_blocks(k_adjoint_f32c<PPL, BLOCK>, BLOCK);
    return v;
}

int adjoint_f32c_blocks_per_cu(int ppl, int block) {
#define SWV_OCC_A(P, B) \
    if (ppl == P && block == B) return adjoint_f32c_occ<P, B>();
    SWV_OCC_A(1, 64) SWV_OCC_A(1, 128) SWV_OCC_A(1, 256)
    SWV_OCC_A(2, 64) SWV_OCC_A(2, 128) SWV_OCC_A(2, 256)
    SWV_OCC_A(4, 64) SWV_OCC_A(4, 128) SWV_OCC_A(4, 256)
#undef SWV_OCC_A
    return 1;
}

// Rows per chunk of the FP64 adjoint and gradients.  Workgroups run in rounds of
// two per CU; up to four rounds rather than one, since the dies' clocks differ, but
// fewer while the partial sums (one set of `bytes` per chunk) exceed 32 MiB, and
// whole rounds: the chunk count is the most that fits r of them.  At least
// kAdjMinRows rows for a wave, so that filling the table stays small beside them,
// and at least 8 chunks of 64 rows and more.
static int64_t cell_chunk(int64_t n_vis, const Columns& C, int64_t bytes, int n_cu) {
    if (n_vis <= 0) return 1;
    const int64_t per_block = C.parts > 1 ? 1 : kAdjWaves;   // (chunk, column) jobs
    const int64_t cols = C.parts > 1 ? 1 : std::max<int64_t>(C.cols, 1);
    const int64_t cap = (int64_t(32) << 20) / std::max<int64_t>(bytes, 1);
    int64_t chunks = 0;
    for (int64_t r = 4; r >= 1; --r) {
        chunks = r * n_cu * 2 * per_block / cols;
        if (chunks <= cap) break;
    }
    chunks = std::max<int64_t>(8, std::min(chunks, cap));
    const int64_t least = (n_vis + chunks - 1) / chunks;
    const int64_t eight = std::max<int64_t>(64, std::max(least, (n_vis + 7) / 8));
    const int64_t chunk = std::min(eight, std::max<int64_t>({64, C.parts * kAdjMinRows, least}));
    return std::min<int64_t>(chunk, int64_t(1) << 30);   // rows per chunk fit an int
}

// Calls too small for four waves on every compute unit run at a wave's latencies,
// which grow with its groups: fewer groups until there are as many waves (100 rows x
// 10,000 pixels, the whole call: 26.8 us with four groups a wave, 17.2 with two, 16.2
// with one, which is the host's time; 1,000 x 30,000, 1,888 waves of four: the same).
int adjoint_cell_groups(int64_t n_vis, int64_t n_pix, int ppl, int n_cu) {
    for (; ppl > 1; ppl /= 2) {
        const Columns C = columns_of(n_pix, ppl);
        const int64_t chunk = adjoint_cell_chunk(n_vis, n_pix, ppl, n_cu);
        const int64_t waves = (n_vis + chunk - 1) / chunk * C.cols * C.parts;
        if (waves >= 4 * (int64_t)n_cu) break;
    }
    return ppl;
}

int64_t adjoint_cell_chunk(int64_t n_vis, int64_t n_pix, int ppl, int n_cu) {
    return cell_chunk(n_vis, columns_of(n_pix, ppl), 16 * n_pix, n_cu);
}

int64_t grad_chunk(int64_t n_vis, int64_t n_comp, int cpl, int n_cu) {
    return cell_chunk(n_vis, columns_of(n_comp, cpl), 32 * n_comp, n_cu);
}

// Workgroups per XCD.
static int64_t cell_run(const Columns& C, int64_t n_chunks) {
    const int64_t blocks = C.parts > 1 || C.cols == kAdjWaves
                               ? n_chunks
                               : (n_chunks * C.cols + kAdjWaves - 1) / kAdjWaves;
    return (blocks + 7) / 8;
}

static hipError_t run_adjoint_cell(hipStream_t s, int ppl, int64_t chunk, int64_t n_vis,
                                   const double* u, const double* v, const double* w,
                                   const void* y, int64_t n_pix, const double* l, const double* m,
                                   const double* nm1, int sign, void* partial) {
    const Columns C = columns_of(n_pix, ppl);
    const int64_t n_chunks = (n_vis + chunk - 1) / chunk, run = cell_run(C, n_chunks);
    if (8 * run > kMaxLaunchThreads / kTabBlock) return hipErrorInvalidConfiguration;
    k_adjoint_cell<<<dim3((unsigned)(8 * run)), dim3(kTabBlock), 0, s>>>(
        u, v, w, (const double2*)y, n_vis, chunk, l, m, nm1, n_pix, (double)sign, C, n_chunks, run,
        (double2*)partial);
    return hipGetLastError();
}

hipError_t launch_adjoint(hipStream_t s, int prec, int ppl, int block, int64_t chunk,
                          int64_t n_vis, const double* u, const double* v, const double* w,
                          const void* y, int64_t n_pix, const double* l, const double* m,
                          const double* nm1, int sign, void* partial, void* out) {
    if (n_pix <= 0) return hipSuccess;
    if (ppl != 1 && ppl != 2 && ppl != 4) return hipErrorInvalidValue;
    const int64_t n_chunks = n_vis > 0 ? (n_vis + chunk - 1) / chunk : 0;
    if (n_chunks > 0 && prec == SWV_FP64) {
        const hipError_t e = run_adjoint_cell(s, ppl, chunk, n_vis, u, v, w, y, n_pix, l, m, nm1,
                                              sign, partial);
        if (e != hipSuccess) return e;
    } else if (n_chunks > 0) {
        const int64_t per_block = (int64_t)block * ppl;
        const int64_t tiles = (n_pix + per_block - 1) / per_block;
#define SWV_RUN_A(P, B)           \
    if (ppl == P && block == B)   \
        run_adjoint_f32c<P, B>(s, tiles, chunk, n_vis, u, v, w, y, n_pix, l, m, nm1, sign, partial);
        SWV_RUN_A(1, 64) SWV_RUN_A(1, 128) SWV_RUN_A(1, 256)
        SWV_RUN_A(2, 64) SWV_RUN_A(2, 128) SWV_RUN_A(2, 256)
        SWV_RUN_A(4, 64) SWV_RUN_A(4, 128) SWV_RUN_A(4, 256)
#undef SWV_RUN_A
        if (block != 64 && block != 128 && block != 256) return hipErrorInvalidValue;
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const auto sum = [&](auto columns) {
        constexpr int COLS = decltype(columns)::value;
        launch_slabs((n_pix + COLS - 1) / COLS, kSumBlock, [&](int64_t b0, unsigned nb) {
            k_sum_chunks_c128<COLS><<<dim3(nb), dim3(kSumBlock), 0, s>>>(
                (const double2*)partial, n_chunks, n_pix, b0, (double2*)out);
        });
    };
    if (n_pix < kSumNarrow)
        sum(std::integral_constant<int, 8>());
    else if (n_chunks <= kSumFew)
        sum(std::integral_constant<int, 256>());
    else
        sum(std::integral_constant<int, 64>());
    return hipGetLastError();
}

// -------------------------------------------------------------- gradients --
// The gradients need four real sums per component k and chunk of rows, with
// z = conj(y) e:
//   Z0 = Re sum z                    (flux:      dchi2/dI ~ Re A^H r)
//   Zu, Zv, Zw = Im sum {u, v, w} z  (positions: d phi/dl = u - w l / n, ...)
// The kernel is the FP64 adjoint's with components for pixels: directions times
// s, conj(y) turned by the rest of the angle, then by the node; Re z goes
// straight into its sum, Im z is formed for the three others.  23 FP64
// instructions per row and component (phase 3, cell 4, rest 5, 4 + 2 + 2 + 3)
// against 32 with the polynomial phasor, bound by their issue.  Rows come by
// scalar loads: staged in LDS as broadcasts they would take as long there as the
// arithmetic does, beside the table's gathers.  261,120 rows x 1,000 components:
// with its prediction and the sums over chunks, 0.53 -> 0.36 ms.
template <int G, bool WIDE>
__device__ __forceinline__ void grad_rows(CellPtr T, const double* u, const double* v,
                                          const double* w, const double2* y, int nrow,
                                          const double (&L)[G], const double (&M)[G],
                                          const double (&N)[G], double (&z)[4][G]) {
    const auto* U = uniform_ptr(u);
    const auto* V = uniform_ptr(v);
    const auto* W = uniform_ptr(w);
    const auto* Y = uniform_ptr(y);
    const CellCoefs K = cell_coefs();
    const auto step = [&](auto rows, int j) {
        constexpr int R = decltype(rows)::value;
        double uj[R], vj[R], wj[R], yr[R], yi[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uj[r] = U[j + r];
            vj[r] = V[j + r];
            wj[r] = W[j + r];
            yr[r] = Y[j + r].x;
            yi[r] = Y[j + r].y;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            Cell e[G];
            double d[G];
#pragma unroll
            for (int i = 0; i < G; ++i)
                e[i] = find_cell<WIDE>(T, fma(uj[r], L[i], fma(vj[r], M[i], wj[r] * N[i])), d[i],
                                       K.magic);
#pragma unroll
            for (int i = 0; i < G; ++i) {
                double cr, sr;
                cell_rest(K, d[i], cr, sr);
                const double tr = fma(cr, yr[r], sr * yi[r]);
                const double ti = fma(sr, yr[r], -(cr * yi[r]));
                z[0][i] = fma(e[i].x, tr, z[0][i]);
                z[0][i] = fma(-e[i].y, ti, z[0][i]);
                const double zi = fma(e[i].x, ti, e[i].y * tr);
                z[1][i] = fma(uj[r], zi, z[1][i]);
                z[2][i] = fma(vj[r], zi, z[2][i]);
                z[3][i] = fma(wj[r], zi, z[3][i]);
            }
        }
    };
    int j = 0;
#pragma unroll 1
    for (; j + kAdjRows <= nrow; j += kAdjRows) step(std::integral_constant<int, kAdjRows>(), j);
#pragma unroll 1
    for (; j < nrow; ++j) step(std::integral_constant<int, 1>(), j);
}

template <int G>
__device__ __forceinline__ void grad_wave(CellPtr T, const double* __restrict__ u,
                                          const double* __restrict__ v,
                                          const double* __restrict__ w,
                                          const double2* __restrict__ y, int nrow, bool wide,
                                          const double* __restrict__ comp, int comp_stride,
                                          int64_t k0, int64_t n_comp, double sgn,
                                          double (&x)[4][4]) {
    double L[G], M[G], N[G], z[4][G];
#pragma unroll
    for (int i = 0; i < G; ++i) {
        int64_t k = k0 + (int64_t)i * 64;
        k = k < n_comp ? k : n_comp - 1;
        L[i] = sgn * comp[k * comp_stride];
        M[i] = sgn * comp[k * comp_stride + 1];
        N[i] = sgn * comp[k * comp_stride + 2];
        z[0][i] = z[1][i] = z[2][i] = z[3][i] = 0.0;
    }
    if (__builtin_expect(wide, 0))
        grad_rows<G, true>(T, u, v, w, y, nrow, L, M, N, z);
    else
        grad_rows<G, false>(T, u, v, w, y, nrow, L, M, N, z);
#pragma unroll
    for (int i = 0; i < G; ++i)
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t][i] = z[t][i];
}

// n_comp_dev, if not null, holds the number of components on the device (a
// captured major cycle whose model changes between replays): the jobs are then
// those of n_comp, the capacity, and waves past the actual count do nothing.
__global__ __launch_bounds__(kTabBlock) __attribute__((amdgpu_waves_per_eu(4))) void k_grad_cell(
    const double* __restrict__ u, const double* __restrict__ v, const double* __restrict__ w,
    const double2* __restrict__ y, int64_t n_vis, int64_t chunk, const double* __restrict__ comp,
    int comp_stride, int64_t n_comp, const int* __restrict__ n_comp_dev, double sgn, Columns C,
    int64_t n_chunks, int64_t run, double* __restrict__ partial) {
    __shared__ Cell T[kTabCells];
    if (n_comp_dev) n_comp = *n_comp_dev;
    WaveJob job = wave_job(n_vis, chunk, C, n_chunks, run);
    if (job.g0 * 64 >= n_comp) job.nrow = 0;
    const bool wide = chunk_is_wide(job, u, v, w);
    fill_cells(T);
    const int64_t j0 = job.j0, k0 = job.g0 * 64 + (threadIdx.x & 63);
    const CellPtr TP = (CellPtr)T;
    double x[4][4] = {};
#define SWV_WAVE(N)                                                                              \
    grad_wave<N>(TP, u + j0, v + j0, w + j0, y + j0, job.nrow, wide, comp, comp_stride, k0, n_comp, \
                 sgn, x)
    switch (job.nrow > 0 ? job.G : 0) {
        case 0: break;
        case 1: SWV_WAVE(1); break;
        case 2: SWV_WAVE(2); break;
        case 3: SWV_WAVE(3); break;
        default: SWV_WAVE(4); break;
    }
#undef SWV_WAVE
    if (!join_parts<4>(T, job, C, x)) return;
    double* part = partial + job.chunk * 4 * n_comp;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int64_t k = k0 + (int64_t)i * 64;
        if (i < job.G && k < n_comp)
#pragma unroll
            for (int t = 0; t < 4; ++t) part[t * n_comp + k] = x[t][i];
    }
}

// A block owns COLS components; thread (q, t, x) adds sum t of component x over
// the chunks q, q + Q, ... in order, then as in the chunk reduction.  8 columns for
// short lists (600 components x 1,536 chunks: 11.3 us, 15.0 with 16), 16 for longer
// ones, whose 64-byte segments cost (2,000 x 1,536: 16.9 us, 30.4 with 8), 64 for the
// longest (100,000 x 64: 30 us, 36 with 16) and for few chunks (1,000,000 x 2: 34 us,
// 270 with 8).
constexpr int kFinishBlock = 1024;

template <int COLS>
__global__ __launch_bounds__(kFinishBlock) void k_grad_finish(
    const double* __restrict__ partial, int64_t n_chunks, const double* __restrict__ comp,
    int comp_stride, int64_t n_comp, const int* __restrict__ n_comp_dev, int64_t bid0, double sgn,
    double alpha, double* __restrict__ d_flux, double* __restrict__ d_l, double* __restrict__ d_m) {
    constexpr int Q = kFinishBlock / (4 * COLS);
    __shared__ double red[Q][4][COLS];
    if (n_comp_dev) n_comp = *n_comp_dev;
    if ((bid0 + blockIdx.x) * COLS >= n_comp) return;   // whole block past the count
    const int tx = threadIdx.x % COLS, t = threadIdx.x / COLS % 4,
              q = threadIdx.x / (4 * COLS);
    const int64_t k = (bid0 + blockIdx.x) * COLS + tx;
    double z = 0.0;
    if (k < n_comp) {
        const double* p = partial + t * n_comp + k;
        int64_t c = q;
        for (; c + (kAhead - 1) * Q < n_chunks; c += kAhead * Q) {
            double x[kAhead];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) x[i] = p[(c + i * Q) * 4 * n_comp];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) z += x[i];
        }
        for (; c < n_chunks; c += Q) z += p[c * 4 * n_comp];
    }
    red[q][t][tx] = z;
    __syncthreads();
    for (int h = Q / 2; h > 0; h >>= 1) {
        if (q < h) red[q][t][tx] += red[q + h][t][tx];
        __syncthreads();
    }
    if (q != 0 || t != 0 || k >= n_comp) return;
    const double z0 = red[0][0][tx], zu = red[0][1][tx], zv = red[0][2][tx], zw = red[0][3][tx];
    const double* c = comp + k * comp_stride;   // l, m, n - 1, I
    const double n = 1.0 + c[2];
    const double f = -alpha * c[3] * sgn * 2.0 * M_PI;
    d_flux[k] = alpha * z0;
    d_l[k] = f * (zu - (c[0] / n) * zw);
    d_m[k] = f * (zv - (c[1] / n) * zw);
}

hipError_t launch_grad(hipStream_t s, int cpl, int64_t chunk, int64_t n_vis, const double* u,
                       const double* v, const double* w, const void* y, const double* comp,
                       int comp_stride, int64_t n_comp, int sign, double alpha, double* partial,
                       double* d_flux, double* d_l, double* d_m, const int* n_comp_dev) {
    if (n_comp <= 0) return hipSuccess;
    if (cpl != 1 && cpl != 2 && cpl != 4) return hipErrorInvalidValue;
    const int64_t n_chunks = n_vis > 0 ? (n_vis + chunk - 1) / chunk : 0;
    if (n_chunks > 0) {
        const Columns C = columns_of(n_comp, cpl);
        const int64_t run = cell_run(C, n_chunks);
        if (8 * run > kMaxLaunchThreads / kTabBlock) return hipErrorInvalidConfiguration;
        k_grad_cell<<<dim3((unsigned)(8 * run)), dim3(kTabBlock), 0, s>>>(
            u, v, w, (const double2*)y, n_vis, chunk, comp, comp_stride, n_comp, n_comp_dev,
            (double)sign, C, n_chunks, run, partial);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const auto finish = [&](auto columns) {
        constexpr int COLS = decltype(columns)::value;
        launch_slabs((n_comp + COLS - 1) / COLS, kFinishBlock, [&](int64_t b0, unsigned nb) {
            k_grad_finish<COLS><<<dim3(nb), dim3(kFinishBlock), 0, s>>>(
                partial, n_chunks, comp, comp_stride, n_comp, n_comp_dev, b0, (double)sign, alpha,
                d_flux, d_l, d_m);
        });
    };
    if (n_comp >= 8192 || n_chunks <= kSumFew)
        finish(std::integral_constant<int, 64>());
    else if (n_comp >= 1024)
        finish(std::integral_constant<int, 16>());
    else
        finish(std::integral_constant<int, 8>());
    return hipGetLastError();
}

// ------------------------------------------------------ residual and chi^2 --
constexpr int kResBlock = 256;
constexpr int kResMaxBlocks = 2048;

int residual_blocks(int64_t n_vis) {
    const int64_t b = (n_vis + kResBlock * 8 - 1) / (kResBlock * 8);
    return (int)(b < 1 ? 1 : (b > kResMaxBlocks ? kResMaxBlocks : b));
}

__global__ __launch_bounds__(kResBlock) void k_residual(const double2* __restrict__ obs,
                                                        const double2* __restrict__ model,
                                                        int64_t n, double2* __restrict__ resid,
                                                        double* __restrict__ partial) {
    __shared__ double red[kResBlock];
    double acc = 0.0;
    const int64_t stride = (int64_t)gridDim.x * kResBlock;
    for (int64_t j = (int64_t)blockIdx.x * kResBlock + threadIdx.x; j < n; j += stride) {
        const double2 a = obs[j], b = model[j];
        const double rr = a.x - b.x, ri = a.y - b.y;
        resid[j] = make_double2(rr, ri);
        acc = fma(rr, rr, fma(ri, ri, acc));
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int h = kResBlock / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// One block: thread t adds partials t, t + kResBlock, ... in order, then a
// fixed binary tree in LDS.
__global__ __launch_bounds__(kResBlock) void k_chi2_finish(const double* __restrict__ partial,
                                                           int nb, double inv_sigma2,
                                                           double* __restrict__ chi2) {
    __shared__ double red[kResBlock];
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += kResBlock) s += partial[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = kResBlock / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *chi2 = red[0] * inv_sigma2;
}

hipError_t launch_residual(hipStream_t s, int64_t n_vis, const void* obs, const void* model,
                           double inv_sigma2, void* resid, double* partial, double* chi2) {
    const int nb = n_vis > 0 ? residual_blocks(n_vis) : 0;
    if (nb > 0) {
        k_residual<<<dim3(nb), dim3(kResBlock), 0, s>>>((const double2*)obs,
                                                        (const double2*)model, n_vis,
                                                        (double2*)resid, partial);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_chi2_finish<<<1, kResBlock, 0, s>>>(partial, nb, inv_sigma2, chi2);
    return hipGetLastError();
}

}  // namespace swv
