// Per-row device code of the direct component sum (section 3.3, Eq. 12),
// shared by the single-instance kernels and the batched ones.
//
// A lane owns VPL visibility rows j[0..VPL) (rows >= limit are computed on a
// clamped index and not stored); every lane of a wave walks the same
// component list, so a component record (l, m, n-1, I; 32 B) is one scalar
// load into SGPRs that enters the FMAs as the scalar operand.  The sum over
// components is a per-lane running sum in a fixed order: bit-reproducible,
// no atomics.
//
// FP64 work per (row, component).  Fewer than kTableMinComp components: phase
// 3 instructions, reduction 2, polynomial phasor 20, MAC 2.  From there on the
// table phasor with the flux folded into the cell polynomials (four products
// per component, at ingest): phase 3, cell 3 + 1, rest 5, and 4 FMAs that turn
// the node straight into the two sums, 16 in all and two register copies per
// component and wave.  2^21 rows x 2,000 components: 3.43 -> 2.22 ms.
//
// The component list is summed in a fixed two-level order that depends on its
// length alone: 8 ranges of A = ceil(n / 8), each in sub-ranges of
// B = max(32, ceil(A / 8)); every sub-range sums from zero, sub-ranges add up
// in order to ranges, ranges to the result.  The kernels that share a row's
// components between waves or workgroups split at those borders, so all of
// them give the same bits, and partial sums stay short.
#pragma once

#include <type_traits>

#include "device_math.h"
#include "launch.h"
#include "phasor_table.h"

namespace swv {

// One packed component: n - 1 = -(l^2 + m^2) / (1 + n), free of cancellation.
// Written with an explicit FMA so every kernel that packs components rounds
// identically.  Sets bits of `bad` for out-of-domain or non-finite input (the
// record is then zero).
__device__ __forceinline__ Comp pack_component(double L, double M, double I, int& bad) {
    const double r2 = fma(L, L, M * M);
    bad = 0;
    if (!(r2 < 1.0)) bad |= kStatusDomain;
    if (!isfinite(L) || !isfinite(M) || !isfinite(I)) bad |= kStatusNonFinite;
    if (bad) return Comp{0.0, 0.0, 0.0, 0.0};
    return Comp{L, M, -r2 / (1.0 + sqrt(1.0 - r2)), I};
}

__device__ __forceinline__ CompF pack_component_f32c(double L, double M, double I, int& bad) {
    const Comp c = pack_component(L, M, I, bad);
    return CompF{c.l, c.m, c.nm1, (float)c.I, 0.0f};
}

__device__ __forceinline__ CompCell pack_component_cell(double L, double M, double I, int& bad) {
    const Comp c = pack_component(L, M, I, bad);
    return comp_cell(c.l, c.m, c.nm1, c.I);
}

using CompCellPtr = const __attribute__((address_space(4))) CompCell*;

// Borders of the summation order.
struct CompRanges {
    int n, A, B;
    // least components of a sub-range, and of a range
    __host__ __device__ explicit CompRanges(int n_comp, int least = 32, int least_range = 1)
        : n(n_comp), A((int)(((int64_t)n_comp + 7) / 8)), B(0) {
        A = A < least_range ? least_range : A;
        B = (A + 7) / 8;
        B = B < least ? least : B;
    }
    // ranges that hold components (the others are empty)
    __host__ __device__ int count() const { return (int)(((int64_t)n + A - 1) / A); }
    // components [begin, end) of range a, sub-range b
    __host__ __device__ int begin(int a, int b) const {
        const int64_t k = (int64_t)a * A + (int64_t)b * B, e = end_of(a);
        return (int)(k < e ? k : e);
    }
    __host__ __device__ int end(int a, int b) const { return begin(a, b + 1); }
    __host__ __device__ int64_t end_of(int a) const {
        const int64_t e = (int64_t)(a + 1) * A;
        return e < n ? e : n;
    }
    // where the sub-range from k0 ends in a range up to `last`; the borders of lists
    // of up to 2^31 - 1 components may not be passed in 32 bits
    __host__ __device__ int next(int k0, int last) const {
        return last - k0 > B ? k0 + B : last;
    }
};

// Copy of a wave-uniform double into a vector register: an FP64 FMA can read
// one scalar operand only, so one coefficient of each two-term polynomial has
// to be a vector.
__device__ __forceinline__ double vector_copy(double s) {
    double v;
    asm("v_mov_b64 %0, %1" : "=v"(v) : "s"(s));
    return v;
}

// re + i im += sum of components [k0, k1).  NB components per step: their
// scalar loads go out together and 4 table gathers or more are in flight
// (scalar and LDS loads share one wait counter, so a load issued ahead would be
// waited for with the next gather anyway).
template <int VPL, bool WIDE, int NB>
__device__ __forceinline__ void component_step(CellPtr T, CompCellPtr cp, int k,
                                               const double (&U)[VPL], const double (&V)[VPL],
                                               const double (&W)[VPL], double (&re)[VPL],
                                               double (&im)[VPL]) {
    CompCell c[NB];
    double Ic1[NB], Is1[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
        c[b] = CompCell{cp[k + b].l,   cp[k + b].m,   cp[k + b].nm1, cp[k + b].I,
                        cp[k + b].Ic0, cp[k + b].Ic1, cp[k + b].Is0, cp[k + b].Is1};
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        Ic1[b] = vector_copy(c[b].Ic1);
        Is1[b] = vector_copy(c[b].Is1);
    }
    double d[NB][VPL];
    Cell e[NB][VPL];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < VPL; ++i)
            e[b][i] = find_cell_by_cells<WIDE>(
                T, fma(U[i], c[b].l, fma(V[i], c[b].m, W[i] * c[b].nm1)), d[b][i]);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            const double q = d[b][i] * d[b][i];
            const double cI = fma(q, fma(q, Ic1[b], c[b].Ic0), c[b].I);
            const double sI = d[b][i] * fma(q, Is1[b], c[b].Is0);
            re[i] = fma(e[b][i].x, cI, re[i]);
            im[i] = fma(e[b][i].y, cI, im[i]);
            re[i] = fma(-e[b][i].y, sI, re[i]);
            im[i] = fma(e[b][i].x, sI, im[i]);
        }
}

template <int VPL, bool WIDE>
__device__ __forceinline__ void add_components(CellPtr T, CompCellPtr cp, int k0, int k1,
                                               const double (&U)[VPL], const double (&V)[VPL],
                                               const double (&W)[VPL], double (&re)[VPL],
                                               double (&im)[VPL]) {
    constexpr int NB = VPL >= 4 ? 1 : 4 / VPL;
    int k = k0;
#pragma unroll 1
    for (; k1 - k >= NB; k += NB) component_step<VPL, WIDE, NB>(T, cp, k, U, V, W, re, im);
    if constexpr (NB > 1) {
#pragma unroll 1
        for (; k < k1; ++k) component_step<VPL, WIDE, 1>(T, cp, k, U, V, W, re, im);
    }
}

// The sums of ranges [a0, a1), handed to put(a, re, im) as each is complete.
template <int VPL, bool WIDE, class Put>
__device__ __forceinline__ void range_sums(CellPtr T, CompCellPtr cp, const CompRanges& R, int a0,
                                           int a1, const double (&U)[VPL], const double (&V)[VPL],
                                           const double (&W)[VPL], Put&& put) {
#pragma unroll 1
    for (int a = a0; a < a1; ++a) {
        double rr[VPL], ri[VPL];
#pragma unroll
        for (int i = 0; i < VPL; ++i) rr[i] = ri[i] = 0.0;
        const int last = (int)R.end_of(a);
#pragma unroll 1
        for (int k0 = a * R.A, k1; k0 < last; k0 = k1) {
            k1 = R.next(k0, last);
            double re[VPL], im[VPL];
#pragma unroll
            for (int i = 0; i < VPL; ++i) re[i] = im[i] = 0.0;
            add_components<VPL, WIDE>(T, cp, k0, k1, U, V, W, re, im);
#pragma unroll
            for (int i = 0; i < VPL; ++i) {
                rr[i] += re[i];
                ri[i] += im[i];
            }
        }
        put(a, rr, ri);
    }
}

// Rows j[0 .. VPL) of a lane, clamped to the last one, times the cells of a turn.
// Returns whether some row of the wave is beyond the cells' direct reach (or not
// finite); the wave's rows are then as they came.
template <int VPL>
__device__ __forceinline__ bool load_rows(const int64_t (&j)[VPL], int64_t limit,
                                          const double* __restrict__ u,
                                          const double* __restrict__ v,
                                          const double* __restrict__ w, double (&U)[VPL],
                                          double (&V)[VPL], double (&W)[VPL]) {
    bool small = true;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        const int64_t jj = j[i] < limit ? j[i] : limit - 1;
        U[i] = u[jj];
        V[i] = v[jj];
        W[i] = w[jj];
        small = small && cells_reach(U[i], V[i], W[i]);
    }
    const bool wide = __any(!small);
    const double scale = wide ? 1.0 : (double)kTabCells;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        U[i] *= scale;
        V[i] *= scale;
        W[i] *= scale;
    }
    return wide;
}

// A visibility in the output's type (the sums are FP64 for either).
__device__ __forceinline__ void store_vis(double2* out, int64_t j, double re, double im) {
    out[j] = make_double2(re, im);
}
__device__ __forceinline__ void store_vis(float2* out, int64_t j, double re, double im) {
    out[j] = make_float2((float)re, (float)im);
}

// All components by one wave; put(j, re, im) stores a row.
template <int VPL, class Put>
__device__ __forceinline__ void direct_rows_cell(CellPtr T, const int64_t (&j)[VPL], int64_t limit,
                                                 const double* __restrict__ u,
                                                 const double* __restrict__ v,
                                                 const double* __restrict__ w,
                                                 const CompCell* __restrict__ comp, int n_comp,
                                                 double sgn, Put&& put,
                                                 int* __restrict__ status) {
    double U[VPL], V[VPL], W[VPL], sr[VPL], si[VPL];
    const bool wide = load_rows<VPL>(j, limit, u, v, w, U, V, W);
#pragma unroll
    for (int i = 0; i < VPL; ++i) sr[i] = si[i] = 0.0;
    const CompRanges R(n_comp);
    const CompCellPtr cp = uniform_ptr(comp);
    const auto add = [&](int, const double(&rr)[VPL], const double(&ri)[VPL]) {
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            sr[i] += rr[i];
            si[i] += ri[i];
        }
    };
    if (__builtin_expect(wide, 0))
        range_sums<VPL, true>(T, cp, R, 0, 8, U, V, W, add);
    else
        range_sums<VPL, false>(T, cp, R, 0, 8, U, V, W, add);
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        if (j[i] < limit) {
            if (!isfinite(U[i] + V[i] + W[i])) atomicOr(status, kStatusNonFinite);
            put(j[i], sr[i], sgn * si[i]);
        }
    }
}

// Rows row0 .. row0 + kTabBlock / SPLIT * VPL of a workgroup, SPLIT waves sharing
// a row's components, 8 / SPLIT ranges each.  Their range sums meet in LDS (where
// the table was: it is gone afterwards) and are added in range order.
template <int VPL, int SPLIT, class Put>
__device__ __forceinline__ void direct_block_cell(Cell* T, int64_t row0, int64_t limit,
                                                  const double* __restrict__ u,
                                                  const double* __restrict__ v,
                                                  const double* __restrict__ w,
                                                  const CompCell* __restrict__ comp, int n_comp,
                                                  double sgn, Put&& put,
                                                  int* __restrict__ status) {
    constexpr int kLanes = kTabBlock / SPLIT;   // lanes that own rows
    constexpr int kRows = kLanes * VPL;         // rows per workgroup
    static_assert(8 * kRows <= kTabCells, "range sums fit where the table was");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = wave % SPLIT, local = wave / SPLIT * 64 + lane;
    int64_t j[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) j[i] = row0 + i * kLanes + local;
    double U[VPL], V[VPL], W[VPL];
    const bool wide = load_rows<VPL>(j, limit, u, v, w, U, V, W);
    const CompRanges R(n_comp);
    constexpr int kOwn = 8 / SPLIT;   // ranges per wave
    double pr[kOwn][VPL], pi[kOwn][VPL];
#pragma unroll
    for (int q = 0; q < kOwn; ++q) {
        const auto keep = [&](int, const double(&re)[VPL], const double(&im)[VPL]) {
#pragma unroll
            for (int i = 0; i < VPL; ++i) {
                pr[q][i] = re[i];
                pi[q][i] = im[i];
            }
        };
        const int a = part * kOwn + q;
        if (__builtin_expect(wide, 0))
            range_sums<VPL, true>((CellPtr)T, uniform_ptr(comp), R, a, a + 1, U, V, W, keep);
        else
            range_sums<VPL, false>((CellPtr)T, uniform_ptr(comp), R, a, a + 1, U, V, W, keep);
    }
    __syncthreads();   // every wave is done with the table
#pragma unroll
    for (int q = 0; q < kOwn; ++q)
#pragma unroll
        for (int i = 0; i < VPL; ++i)
            T[(part * kOwn + q) * kRows + i * kLanes + local] = Cell{pr[q][i], pi[q][i]};
    __syncthreads();
    for (int r = threadIdx.x; r < kRows && row0 + r < limit; r += kTabBlock) {
        double re = 0.0, im = 0.0;
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const Cell p = T[a * kRows + r];
            re += p.x;
            im += p.y;
        }
        const int64_t jr = row0 + r;
        if (!isfinite(u[jr] + v[jr] + w[jr])) atomicOr(status, kStatusNonFinite);
        put(jr, re, sgn * im);
    }
}

// Polynomial phasor, components in list order; comp: records in any address space.
template <int VPL, class RecPtr, class Put>
__device__ __forceinline__ void direct_rows_f64(const int64_t (&j)[VPL], int64_t limit,
                                                const double* __restrict__ u,
                                                const double* __restrict__ v,
                                                const double* __restrict__ w,
                                                RecPtr comp, int n_comp,
                                                double sgn, Put&& put, int* __restrict__ status) {
    double U[VPL], V[VPL], W[VPL], re[VPL], iq[VPL];
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        const int64_t jj = j[i] < limit ? j[i] : limit - 1;
        U[i] = u[jj];
        V[i] = v[jj];
        W[i] = w[jj];
        re[i] = 0.0;
        iq[i] = 0.0;
    }
    for (int k = 0; k < n_comp; ++k) {
        const Comp cur{comp[k].l, comp[k].m, comp[k].nm1, comp[k].I};
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            double c, q;
            cis2pi_q(reduced_phase(U[i], V[i], W[i], cur.l, cur.m, cur.nm1), c, q);
            re[i] = fma(cur.I, c, re[i]);
            iq[i] = fma(cur.I, q, iq[i]);
        }
    }
    const double s4 = 4.0 * sgn;
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        if (j[i] < limit) {
            if (!isfinite(U[i] + V[i] + W[i])) atomicOr(status, kStatusNonFinite);
            put(j[i], re[i], s4 * iq[i]);
        }
    }
}

// FP32-compensated form: FP64 phase, reduced to [-1/2, 1/2] turns exactly; FP32
// phasor, products and Kahan sums.  Components come in fours: their products and
// the running compensation meet in a chain of FMAs, then one Kahan step, so a
// component costs a quarter of a step (the chain's roundings stay within a few
// 2^-24 of the four terms); then a pair and a single one.  Per row and component 5
// FP64 instructions and the conversion for the phase, the hardware sine and cosine,
// 3.5 FP32 for the sums.  1,263,601 rows x 1,999 components: 0.90 ms.
//
// The reduction is exact for every baseline and direction, those behind the phase
// centre's horizon too, and a phase near zero, of either sign, keeps FP32's relative
// accuracy.  Reduced to [0, 1) by the hardware fract, one instruction less, it takes
// 0.83 ms, but rounds by up to 2^-25 turns instead of 2^-26 (4.2e-9 of the flux
// against 3.4e-9 rms, 2,000 components, 1e5 wavelengths) and negative phases near
// zero not relatively at all; summed onto a magic number whose last place is a
// fixed fraction of a turn, 0.80 ms, but right only as far as that number's range
// goes.
//
// The list is summed in the FP64 kernels' two-level order with sub-ranges of at
// least kF32cSub components and ranges of at least kF32cRange; their compensated
// sums enter the ranges' and the total in FP64.  A range costs a row eight FP64
// additions and conversions, so short lists are cut into few of them: 10,000,000 rows
// x 32 components in 8, 2 and 1 ranges 161, 129 and 125 us, x 128 in 8, 4 and 2 450,
// 437 and 429.  A list of one range keeps its sums in FP32 to the end (x 32: 119 us),
// the same bits.
constexpr int kF32cSub = 128, kF32cRange = 64;

// Sums s and compensations c of components [k0, k1).
template <int VPL, class CompPtr>
__device__ __forceinline__ void sum_components_f32c(CompPtr cp, int k0, int k1,
                                                    const double (&U)[VPL], const double (&V)[VPL],
                                                    const double (&W)[VPL], float (&sr)[VPL],
                                                    float (&si)[VPL], float (&cr)[VPL],
                                                    float (&ci)[VPL]) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) sr[i] = cr[i] = si[i] = ci[i] = 0.0f;
    const auto step = [&](auto count, int k) {
        constexpr int N = decltype(count)::value;
        CompF c[N];
#pragma unroll
        for (int b = 0; b < N; ++b)
            c[b] = CompF{cp[k + b].l, cp[k + b].m, cp[k + b].nm1, cp[k + b].I, 0.0f};
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            float yr = -cr[i], yi = -ci[i];
#pragma unroll
            for (int b = N - 1; b >= 0; --b) {
                float co, sn;
                cis2pi_f32((float)reduced_phase(U[i], V[i], W[i], c[b].l, c[b].m, c[b].nm1), co, sn);
                yr = fmaf(c[b].I, co, yr);
                yi = fmaf(c[b].I, sn, yi);
            }
            kahan_step(yr, sr[i], cr[i]);
            kahan_step(yi, si[i], ci[i]);
        }
    };
    int k = k0;
#pragma unroll 1
    for (; k1 - k >= 4; k += 4) step(std::integral_constant<int, 4>(), k);
    if (k1 - k >= 2) {
        step(std::integral_constant<int, 2>(), k);
        k += 2;
    }
    if (k < k1) step(std::integral_constant<int, 1>(), k);
}

// Their sums added to re + i im.
template <int VPL, class CompPtr>
__device__ __forceinline__ void add_components_f32c(CompPtr cp, int k0, int k1,
                                                    const double (&U)[VPL], const double (&V)[VPL],
                                                    const double (&W)[VPL],
                                                    double (&re)[VPL], double (&im)[VPL]) {
    float sr[VPL], si[VPL], cr[VPL], ci[VPL];
    sum_components_f32c<VPL>(cp, k0, k1, U, V, W, sr, si, cr, ci);
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        re[i] += (double)sr[i] - (double)cr[i];
        im[i] += (double)si[i] - (double)ci[i];
    }
}

// The sums of ranges [a0, a1), handed to put(a, re, im) as each is complete.
template <int VPL, class CompPtr, class Put>
__device__ __forceinline__ void range_sums_f32c(CompPtr cp, const CompRanges& R, int a0, int a1,
                                                const double (&U)[VPL], const double (&V)[VPL],
                                                const double (&W)[VPL], Put&& put) {
#pragma unroll 1
    for (int a = a0; a < a1; ++a) {
        double rr[VPL], ri[VPL];
#pragma unroll
        for (int i = 0; i < VPL; ++i) rr[i] = ri[i] = 0.0;
        const int last = (int)R.end_of(a);
#pragma unroll 1
        for (int k0 = a * R.A, k1; k0 < last; k0 = k1) {
            k1 = R.next(k0, last);
            add_components_f32c<VPL>(cp, k0, k1, U, V, W, rr, ri);
        }
        put(a, rr, ri);
    }
}

// Rows j[0 .. VPL) of a lane, clamped to the last one.
template <int VPL>
__device__ __forceinline__ void load_rows_f32c(const int64_t (&j)[VPL], int64_t limit,
                                               const double* __restrict__ u,
                                               const double* __restrict__ v,
                                               const double* __restrict__ w, double (&U)[VPL],
                                               double (&V)[VPL], double (&W)[VPL]) {
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        const int64_t jj = j[i] < limit ? j[i] : limit - 1;
        U[i] = u[jj];
        V[i] = v[jj];
        W[i] = w[jj];
    }
}

template <int VPL>
__device__ __forceinline__ void direct_rows_f32c(const int64_t (&j)[VPL], int64_t limit,
                                                 const double* __restrict__ u,
                                                 const double* __restrict__ v,
                                                 const double* __restrict__ w,
                                                 const CompF* __restrict__ comp, int n_comp,
                                                 double sgn, float2* __restrict__ out,
                                                 int* __restrict__ status) {
    double U[VPL], V[VPL], W[VPL], sr[VPL], si[VPL];
    load_rows_f32c<VPL>(j, limit, u, v, w, U, V, W);
    if (n_comp <= kF32cRange) {
        float fr[VPL], fi[VPL], cr[VPL], ci[VPL];
        sum_components_f32c<VPL>(uniform_ptr(comp), 0, n_comp, U, V, W, fr, fi, cr, ci);
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            if (j[i] < limit) {
                if (!isfinite(U[i] + V[i] + W[i])) atomicOr(status, kStatusNonFinite);
                out[j[i]] = make_float2(fr[i] - cr[i], (float)sgn * (fi[i] - ci[i]));
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < VPL; ++i) sr[i] = si[i] = 0.0;
    const CompRanges R(n_comp, kF32cSub, kF32cRange);
    const auto add = [&](int, const double(&rr)[VPL], const double(&ri)[VPL]) {
#pragma unroll
        for (int i = 0; i < VPL; ++i) {
            sr[i] += rr[i];
            si[i] += ri[i];
        }
    };
    range_sums_f32c<VPL>(uniform_ptr(comp), R, 0, R.count(), U, V, W, add);
#pragma unroll
    for (int i = 0; i < VPL; ++i) {
        if (j[i] < limit) {
            if (!isfinite(U[i] + V[i] + W[i])) atomicOr(status, kStatusNonFinite);
            store_vis(out, j[i], sr[i], sgn * si[i]);
        }
    }
}

}  // namespace swv
