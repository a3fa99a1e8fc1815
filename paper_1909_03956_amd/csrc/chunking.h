// Block order of the row-chunked kernels (1-D grid): workgroups are dealt to
// the 8 XCDs round-robin by linear id, and blocks sharing a chunk read the same
// rows.  Ids therefore walk groups of 8 chunks -- one per XCD -- and, inside a
// group, all tiles in consecutive dispatch rounds: every tile of a chunk runs
// on the same XCD at about the same time and the chunk's rows come from HBM
// into one L2 once.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace swv {

// Chunk count rounded up to a whole number of XCD rounds.
inline int64_t xcd_padded(int64_t n_chunks) { return (n_chunks + 7) / 8 * 8; }

// (chunk, tile) of linear block id `bid` in the order described above.
__device__ __forceinline__ void chunk_tile(int64_t bid, int64_t tiles, int64_t& chunk,
                                           int64_t& tile) {
    const int64_t per_group = 8 * tiles;
    const int64_t g = bid / per_group;
    const int64_t r = bid - g * per_group;
    tile = r >> 3;
    chunk = g * 8 + (r & 7);
}

// HIP takes no launch of 2^32 threads or more in a dimension; kernels that would
// need more go out in slabs of half that.
constexpr int64_t kMaxLaunchThreads = int64_t(1) << 31;

// Launches `total` blocks of `block` threads as 1-D grids of one slab each, passing
// the first linear id of each.
template <class F>
static void launch_slabs(int64_t total, int block, F&& launch) {
    const int64_t slab = kMaxLaunchThreads / block;
    for (int64_t b0 = 0; b0 < total; b0 += slab)
        launch(b0, (unsigned)(total - b0 < slab ? total - b0 : slab));
}

// Rows of one launch of the kernels that give a row up to eight threads.
constexpr int64_t kRowSlab = kMaxLaunchThreads / 8;

// Calls launch(first row, rows) for slabs of that many rows; the first error.
template <class F>
static hipError_t launch_row_slabs(int64_t n, F&& launch) {
    hipError_t e = hipSuccess;
    for (int64_t j = 0; j < n && e == hipSuccess; j += kRowSlab)
        e = launch(j, n - j < kRowSlab ? n - j : kRowSlab);
    return e;
}

}  // namespace swv
