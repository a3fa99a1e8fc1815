// Internal definitions shared by the host runtime and the kernels of libswvis.
#pragma once

#include <cstdint>
#include <string>

#include "../../include/swvis.h"

namespace swv {

// One packed component as the direct kernels read it: 32 bytes, so a wave
// fetches a whole record with one scalar load.  nm1 = n - 1.
struct alignas(32) Comp {
    double l, m, nm1, I;
};

// The same for the FP32-compensated direct kernels: their products take I in FP32.
struct alignas(32) CompF {
    double l, m, nm1;
    float I, unused;
};

// One packed component of the FP64 direct kernels (64 bytes): the same, and the
// coefficients of the phasor inside a table cell times the flux.
struct alignas(64) CompCell {
    double l, m, nm1, I, Ic0, Ic1, Is0, Is1;
};

// One record of the depth-first tree stream (32 bytes, host).
//   root : a = A_1 * lambda_1 of the level-1 node that follows; meta = 0
//   node : a, b, c = h^0, h^1, h^2 with h^m = s^m_{c0} gamma^m_j (sqrt(A_j)/4) 4^-(J-j-1),
//          c0 the node's first child, s the Eq. 10 signs (a thresholded tree:
//          0 for a coefficient that is not kept)
//   leaf : a, b, c = l, m, n - 1 of the pixel centre
// meta of nodes and leaves:
//   bits 0-3   child mask (bit c set if child 4k + c exists; 0 for a leaf)
//   bits 8-12  level j
struct alignas(32) TRec {
    double a, b, c;
    unsigned long long meta;
};

constexpr unsigned meta_mask(unsigned long long meta) { return (unsigned)(meta & 0xFu); }
constexpr int meta_level(unsigned long long meta) { return (int)((meta >> 8) & 31u); }
constexpr unsigned long long make_meta(unsigned mask, int level) {
    return (unsigned long long)(mask & 0xFu) | ((unsigned long long)level << 8);
}

// Deferred-error bits the kernels raise in the context's status word.
enum : int { kStatusDomain = 1, kStatusNonFinite = 2 };

// Sets the thread-local message and returns `code`.
int fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
void clear_error();

}  // namespace swv
