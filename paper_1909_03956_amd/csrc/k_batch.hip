// Batched prediction: many instances (channels x pointings) of uneven size in
// one launch for the FP64 ones (direct sums and trees' leaf sums) and one for the
// FP32-compensated.
//
// The host splits every instance into row tiles and orders the (instance, tile)
// work items by decreasing cost, largest first, so long and short instances
// balance across the chip.  FP64: a workgroup per item, dealt by the hardware.
// FP32-compensated: each wave of a grid sized to stay resident takes the next
// item from a device counter (one atomic per item, on lane 0) and leaves when the
// counter passes the item count, so every wave exits.  The row arithmetic is the
// single-instance kernels' (direct_rows.h).
#include "chunking.h"
#include "direct_rows.h"

namespace swv {

// Packs the components of every direct instance: block row y is instance y.
__global__ void k_batch_ingest(const BatchInst* __restrict__ inst, int* __restrict__ status) {
    const BatchInst I = inst[blockIdx.y];
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (I.is_tree || k >= I.n_comp) return;
    int bad;
    CompCell* own = I.comp;
    if (I.prec == SWV_FP64)
        own[k] = pack_component_cell(I.l[k], I.m[k], I.flux[k], bad);
    else
        ((CompF*)own)[k] = pack_component_f32c(I.l[k], I.m[k], I.flux[k], bad);
    if (bad) atomicOr(status, bad);
}

hipError_t launch_batch_ingest(hipStream_t s, const BatchInst* inst, int n_inst, int max_comp,
                               int* status) {
    if (n_inst <= 0 || max_comp <= 0) return hipSuccess;
    k_batch_ingest<<<dim3((unsigned)((max_comp + 255) / 256), (unsigned)n_inst), dim3(256), 0,
                     s>>>(inst, status);
    return hipGetLastError();
}

// Work-counter reset as a kernel, so a captured graph re-arms itself on
// every replay without a memset node.
__global__ void k_reset_counters(unsigned* counters, int n) {
    if ((int)threadIdx.x < n) counters[threadIdx.x] = 0u;
}

hipError_t launch_reset_counters(hipStream_t s, unsigned* counters, int n) {
    k_reset_counters<<<1, 64, 0, s>>>(counters, n);
    return hipGetLastError();
}

__device__ __forceinline__ unsigned next_item(unsigned* counter) {
    unsigned it = 0;
    if ((threadIdx.x & 63) == 0) it = atomicAdd(counter, 1u);
    return __builtin_amdgcn_readfirstlane(it);
}

// FP64 items.  An item is either whole rows per wave, kBatchRows at a time, or
// kBatchSplitRows rows whose components all eight waves share (short work for the
// chip, long lists).  Lists too short for the table kernels go through the
// polynomial phasor, as in the single-instance call, so the bits are the same.
__global__ __launch_bounds__(kTabBlock) __attribute__((amdgpu_waves_per_eu(4))) void
k_batch_direct(const BatchInst* __restrict__ inst, const WorkItem* __restrict__ items,
               int* __restrict__ status) {
    __shared__ Cell T[kTabCells];
    const auto* it = uniform_ptr(items) + blockIdx.x;
    const auto* I = uniform_ptr(inst) + it->inst;
    const int64_t row0 = it->row0, n_vis = I->n_vis;
    const int64_t limit = row0 + it->nrows < n_vis ? row0 + it->nrows : n_vis;
    const double* u = I->u;
    const double* v = I->v;
    const double* w = I->w;
    void* out = I->out;
    const CompCell* comp = I->comp;
    const int n_comp = I->n_comp;
    const double sgn = I->sgn;
    const bool single = I->prec == SWV_F32C;   // a tree with complex64 output
    const auto put = [out, single](int64_t j, double re, double im) {
        if (single)
            store_vis((float2*)out, j, re, im);
        else
            store_vis((double2*)out, j, re, im);
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (n_comp < kTableMinComp) {
        for (int64_t r = row0 + threadIdx.x; r < limit; r += kTabBlock) {
            const int64_t j[1] = {r};
            direct_rows_f64<1>(j, limit, u, v, w, uniform_ptr((const CompCell*)comp), n_comp, sgn,
                               put, status);
        }
        return;
    }
    fill_cells(T);
    if (it->split) {
        direct_block_cell<4, 8>(T, row0, limit, u, v, w, comp, n_comp, sgn, put, status);
        return;
    }
    for (int64_t r = row0 + wave * 256; r < limit; r += kBatchRows) {
        int64_t j[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) j[i] = r + i * 64 + lane;
        direct_rows_cell<4>((CellPtr)T, j, limit, u, v, w, comp, n_comp, sgn, put, status);
    }
}

// F32C items.
__global__ __launch_bounds__(kBatchF32Block) void k_batch_direct_f32c(
    const BatchInst* __restrict__ inst, const WorkItem* __restrict__ items, unsigned n_items,
    unsigned* __restrict__ counter, int* __restrict__ status) {
    const int lane = threadIdx.x & 63;
    const auto* IT = uniform_ptr(items);
    const auto* IN = uniform_ptr(inst);
    for (;;) {
        const unsigned it = next_item(counter);
        if (it >= n_items) break;
        const int64_t row0 = IT[it].row0;
        const int nrows = IT[it].nrows;
        const int ii = IT[it].inst;
        const int64_t n_vis = IN[ii].n_vis;
        const int64_t limit = row0 + nrows < n_vis ? row0 + nrows : n_vis;
        const double* u = IN[ii].u;
        const double* v = IN[ii].v;
        const double* w = IN[ii].w;
        float2* out = (float2*)IN[ii].out;
        const CompF* comp = (const CompF*)IN[ii].comp;
        const int n_comp = IN[ii].n_comp;
        const double sgn = IN[ii].sgn;
        for (int sub = 0; sub < nrows; sub += 64 * kBatchF32Vpl) {
            int64_t j[kBatchF32Vpl];
#pragma unroll
            for (int i = 0; i < kBatchF32Vpl; ++i) j[i] = row0 + sub + i * 64 + lane;
            direct_rows_f32c<kBatchF32Vpl>(j, limit, u, v, w, comp, n_comp, sgn, out, status);
        }
    }
}

template <class K>
static int resident(K kernel, int block) {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, block, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return nb > 0 ? nb : 1;
}

bool batch_split(int64_t total_rows, int64_t n_comp, int n_cu) {
    return n_comp >= 500 || total_rows < 4 * (int64_t)kBatchRows * 2 * n_cu;
}

int batch_item_rows(int64_t total_rows, int64_t n_comp, int n_cu) {
    if (batch_split(total_rows, n_comp, n_cu)) return kBatchSplitRows;
    const int64_t rounds = total_rows / ((int64_t)kBatchRows * 2 * n_cu);
    return kBatchRows * (int)(rounds >= 32 ? (rounds >= 512 ? 16 : rounds / 32) : 1);
}

int batch_direct_f32c_blocks_per_cu() { return resident(k_batch_direct_f32c, kBatchF32Block); }

hipError_t launch_batch_direct(hipStream_t s, const BatchInst* inst, const WorkItem* items,
                               unsigned n_items, int* status) {
    launch_slabs(n_items, kTabBlock, [&](int64_t i0, unsigned n) {
        k_batch_direct<<<dim3(n), dim3(kTabBlock), 0, s>>>(inst, items + i0, status);
    });
    return hipGetLastError();
}

hipError_t launch_batch_direct_f32c(hipStream_t s, int grid, const BatchInst* inst,
                                    const WorkItem* items, unsigned n_items, unsigned* counter,
                                    int* status) {
    if (n_items == 0) return hipSuccess;
    k_batch_direct_f32c<<<dim3(grid), dim3(kBatchF32Block), 0, s>>>(inst, items, n_items, counter,
                                                                    status);
    return hipGetLastError();
}

}  // namespace swv
