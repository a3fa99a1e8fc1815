// exp(2 pi i phi) from a table of 4,096 cells in LDS: the node's phasor
// (cos, sin)(2 pi k / 4096), correctly rounded, turned by the small angle left
// over, whose sine and cosine take two polynomial terms each.
//
// Why a table: the polynomial phasor of device_math.h costs 20 FP64
// instructions of the 27 per term of the direct sum, and the kernels are bound
// by VALU issue (every VALU instruction, 32-bit ones too, was measured at
// 0.8-1.0 of an FP64 FMA's issue slot).  A cell lookup leaves, after the phase:
// 3 to find the node and the rest (one addition of 1.5 2^40 puts the node's
// number in the low mantissa bits), 1 for the LDS offset, 5 for the
// polynomials and 4 to turn the node.  The gather itself runs beside the VALU:
// one ds_read_b128 at random cells takes 11.4 cycles per wave and CU, under
// the 16-20 issue slots around it.
//
// Why 4,096 cells: the rest is at most 1/8192 turn, so two terms each keep the
// polynomials' error (1.5e-19) far below rounding; and a 16-bit shift
// (v_lshlrev_b16, upper half zero) then is index modulo 4,096 and byte offset
// in one instruction.  512 cells with three-term sines took 2.56 ms, 2,048
// cells 2.30 ms and 4,096 cells 2.22 ms on 2^21 rows x 2,000 components
// (3.43 ms with the polynomial phasor).  The table takes 64 KB, so its kernels
// run 512-thread workgroups, two to a CU.
//
// Error: the node's rounding (2^-54) and two roundings of the turned value,
// against about five roundings in the polynomial phasor's double-angle steps.
#pragma once

#include <hip/hip_runtime.h>

#include "device_math.h"
#include "launch.h"
#include "sincos_table.h"

namespace swv {

constexpr int kTabCells = 4096;
// 1.5 2^52 / kTabCells: adding it rounds to a whole cell, whose number modulo
// 2^32 is then the low word.  Exact for |phase| < 2^39; larger phases go
// through the WIDE form, which takes off whole turns first.
constexpr double kTabMagic = 1.5 * 0x1p40;
// Rows whose |u| + |v| + |w| stays below this have |phase| < 2^39 for every
// direction with |l|, |m|, |n - 1| <= 2.
constexpr double kTabMaxBaseline = 0x1p38;
__device__ __forceinline__ bool cells_reach(double u, double v, double w) {
    return fabs(u) + fabs(v) + fabs(w) < kTabMaxBaseline;
}

typedef double Cell __attribute__((ext_vector_type(2)));
using CellPtr = const __attribute__((address_space(3))) Cell*;

// Fills the workgroup's table and waits for it.  From the first octant: the
// angles at j cells to either side of each axis.
__device__ __forceinline__ void fill_cells(Cell* T) {
    for (int j = threadIdx.x; j <= 512; j += blockDim.x) {
        const double c = kOctant[j][0], s = kOctant[j][1];
        T[j] = Cell{c, s};
        T[1024 + j] = Cell{-s, c};
        T[2048 + j] = Cell{-c, -s};
        T[3072 + j] = Cell{s, -c};
        if (j > 0 && j < 512) {   // each cell is written once
            T[1024 - j] = Cell{s, c};
            T[2048 - j] = Cell{-c, s};
            T[3072 - j] = Cell{-s, -c};
            T[4096 - j] = Cell{c, -s};
        }
    }
    __syncthreads();
}

// The cell polynomials' coefficients and the magic number as vector registers,
// for kernels whose records do not carry them: an FP64 FMA reads one scalar
// operand only, and the compiler would copy one of two constants for every use.
struct CellCoefs {
    double c0, c1, s0, s1, magic;
};
__device__ __forceinline__ CellCoefs cell_coefs() {
    return CellCoefs{vector_const(kCellC[0]), vector_const(kCellC[1]), vector_const(kCellS[0]),
                     vector_const(kCellS[1]), vector_const(kTabMagic)};
}

// Cell of a phase in turns and the rest d (turns, |d| <= 1/8192).  The phase
// minus the node is exact.  WIDE takes whole turns off first, exactly, which
// leaves the same cell and the same d wherever both forms apply (a whole turn
// is an even number of cells, so ties round alike); non-finite phases give
// NaN and some cell of the table.
template <bool WIDE>
__device__ __forceinline__ Cell find_cell(CellPtr T, double phase, double& d,
                                          double magic = kTabMagic) {
    const double r = WIDE ? phase - rint(phase) : phase;
    const double t = r + magic;
    d = r - (t - magic);
    unsigned off;
    // 16-bit shift: (low word mod 4096) * 16, upper half zero
    asm("v_lshlrev_b16_e32 %0, 4, %1" : "=v"(off) : "v"((unsigned)__double_as_longlong(t)));
    return *(CellPtr)((const __attribute__((address_space(3))) char*)T + off);
}

// (cos, sin)(2 pi d) of the rest.
__device__ __forceinline__ void cell_rest(const CellCoefs& K, double d, double& c, double& s) {
    const double q = d * d;
    c = fma(q, fma_v(q, K.c1, K.c0), 1.0);
    s = d * fma_v(q, K.s1, K.s0);
}

// a b + c with a a scalar register (wave-uniform).
__device__ __forceinline__ double fma_s(double a, double b, double c) {
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "s"(a), "v"(b), "v"(c));
    return d;
}

// The same of the phase a b, which is never rounded at its own magnitude: one
// rounding to the cell, one of the rest.  a is wave-uniform.
template <bool WIDE>
__device__ __forceinline__ Cell find_cell_product(CellPtr T, double a, double b, double magic,
                                                  double& d) {
    double t;
    if constexpr (WIDE) {
        const double p = a * b;
        const double r = (p - rint(p)) + fma(a, b, -p);   // may exceed half a turn
        const double r1 = r - rint(r);
        t = r1 + magic;
        d = r1 - (t - magic);
    } else {
        t = fma_s(a, b, magic);
        d = fma(a, b, -(t - magic));
    }
    unsigned off;
    asm("v_lshlrev_b16_e32 %0, 4, %1" : "=v"(off) : "v"((unsigned)__double_as_longlong(t)));
    return *(CellPtr)((const __attribute__((address_space(3))) char*)T + off);
}

// The direct sums' form: phases and rests in cells instead of turns (rows times
// 4,096, exactly, so every bit is the other form's), which keeps the coefficients
// below 1 in magnitude: their products with a flux stay finite up to the largest
// one.  WIDE takes the phase in turns.
constexpr double kCellTurns = 1.0 / kTabCells;
constexpr double kCellMagic = kTabMagic * kTabCells;
template <bool WIDE>
__device__ __forceinline__ Cell find_cell_by_cells(CellPtr T, double phase, double& d) {
    const double r = WIDE ? (phase - rint(phase)) * kTabCells : phase;
    const double t = r + kCellMagic;
    d = r - (t - kCellMagic);
    unsigned off;
    asm("v_lshlrev_b16_e32 %0, 4, %1" : "=v"(off) : "v"((unsigned)__double_as_longlong(t)));
    return *(CellPtr)((const __attribute__((address_space(3))) char*)T + off);
}

// A component with its flux times the polynomials' coefficients of rests in cells.
__host__ __device__ __forceinline__ CompCell comp_cell(double l, double m, double nm1, double I) {
    constexpr double c = kCellTurns, c2 = c * c;
    return CompCell{l,
                    m,
                    nm1,
                    I,
                    I * (kCellC[0] * c2),
                    I * (kCellC[1] * c2 * c2),
                    I * (kCellS[0] * c),
                    I * (kCellS[1] * c * c2)};
}

}  // namespace swv
