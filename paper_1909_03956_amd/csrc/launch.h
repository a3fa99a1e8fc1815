// Host-side launchers of the gfx950 kernels (internal to libswvis).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

#include "common.h"

namespace swv {

// Reads through the constant address space: a wave-uniform index then
// compiles to a scalar (SMEM) load whose result lands in SGPRs and feeds
// every lane's arithmetic for free.  Only for memory no kernel writes while
// the reading kernel runs.
template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* uniform_ptr(const T* p) {
    return (const __attribute__((address_space(4))) T*)p;
}

// Tile shapes compiled for each kernel family.
constexpr int kPerLaneOptions[3] = {1, 2, 4};
constexpr int kBlockOptions[3] = {64, 128, 256};

// Threads of the workgroups that share a phasor table in LDS (phasor_table.h).
constexpr int kTabBlock = 512;

hipError_t launch_ingest(hipStream_t s, int64_t n, const double* l, const double* m,
                         const double* flux, Comp* out, int* status);
hipError_t launch_ingest(hipStream_t s, int64_t n, const double* l, const double* m,
                         const double* flux, CompF* out, int* status);
hipError_t launch_ingest(hipStream_t s, int64_t n, const double* l, const double* m,
                         const double* flux, CompCell* out, int* status);

// Shortest component list of the FP64 kernels with the table phasor.  Below
// it the sum is bound by the rows' 40 bytes (at 8 components their transfer
// and the polynomial phasors take about the same time), and filling the table
// (64 KB per workgroup) would cost more than it saves.
constexpr int kTableMinComp = 16;

// FP64 direct sum of fewer than kTableMinComp components, packed in the kernel.
hipError_t launch_direct_few(hipStream_t s, int64_t n_vis, const double* u, const double* v,
                             const double* w, int n_comp, const double* l, const double* m,
                             const double* flux, int sign, double2* out, int* status);

// How the table kernels lay out one call: rows per lane, waves of a workgroup
// that share a row's components (1, 2, 4, 8), and workgroups that share them
// besides (1 or 8, through partial sums in memory).  Every layout gives the
// same bits.
struct DirectShape {
    int vpl = 1, split = 1, parts = 1;
};
// FP32-compensated direct sum; (vpl, block) where no components are shared.
// partials: whether workgroups may share components too.
DirectShape direct_shape_f32c(int64_t n_vis, int64_t n_comp, int n_cu, bool partials);
hipError_t launch_direct_f32c(hipStream_t s, const DirectShape& sh, int vpl, int block,
                              int64_t n_vis, const double* u, const double* v, const double* w,
                              const CompF* comp, int64_t n_comp, int sign, void* out,
                              double2* partial, int* status);

// vpl_max: most rows per lane (1, 2, 4).
DirectShape direct_shape(int64_t n_vis, int64_t n_comp, int vpl_max, int n_cu, bool partials);
// Bytes of partial sums that hold any launch of these shapes: the most rows whose
// components workgroups share are 64 per compute unit (FP64: half of that).
inline size_t direct_partial_bytes(int n_cu) { return 64 * sizeof(double2) * 64 * (size_t)n_cu; }
// FP64 direct sum of packed components (fewer than kTableMinComp: polynomial
// phasor, whatever the layout); prec is that of the output alone (SWV_F32C:
// complex64).
hipError_t launch_direct_cell(hipStream_t s, const DirectShape& sh, int64_t n_vis, const double* u,
                              const double* v, const double* w, const CompCell* comp,
                              int64_t n_comp, int sign, int prec, void* out, double2* partial,
                              int* status);

// Limits of the trees the entry points predict: levels up to kTreeMaxJ, or at
// any level fewer than kTreeMaxSeg branching nodes on a root-to-leaf path; a
// record stream that 32-bit byte offsets address.  The leaf sum has none of them:
// they are the interface's, which refuses what it always has.
constexpr int kTreeMaxJ = 16;
constexpr int kTreeMaxSeg = 16;
constexpr size_t kMaxRecordBytes = 0xFFFFFFE0u;

// ppl: FP64 the most 64-pixel groups per wave, F32C pixels per lane; block: F32C
// threads per workgroup (the FP64 form's workgroups share a phasor table and
// have a size of their own).
hipError_t launch_adjoint(hipStream_t s, int prec, int ppl, int block, int64_t chunk,
                          int64_t n_vis, const double* u, const double* v, const double* w,
                          const void* y, int64_t n_pix, const double* l, const double* m,
                          const double* nm1, int sign, void* partial, void* out);

// Dirty images on a regular grid by axis phasors (k_grid_image.hip): quads of
// pixels (+-l, +-m), l = (kx0 + i) cell for i < Kx, m alike.
struct GridGeom {
    int kx0, Kx, ky0, Ky;
    double cell;
    __host__ __device__ double r2(int i, int k) const {
        const double l = (double)(kx0 + i) * cell, m = (double)(ky0 + k) * cell;
        return l * l + m * m;
    }
    __host__ __device__ bool on_disk(int i, int k) const { return r2(i, k) < 1.0; }
    __host__ __device__ double nm1(int i, int k) const {
        const double t = r2(i, k);
        return t < 1.0 ? -t / (1.0 + sqrt(1.0 - t)) : 0.0;
    }
};
// Quads with lanes along x (along y if swapped).
struct GridRegion {
    int lane0, lane_n, step0, step_n;
    bool swapped;
};
// How waves cover the quads: octets and diagonal blocks of the square of whole 64
// x 64 blocks, then up to three regions beside it.
struct GridPlan {
    int64_t oct_jobs = 0, diag_jobs = 0, region_jobs[3] = {0, 0, 0}, jobs = 0;
    int step = 0;   // step positions of a region's job
    GridRegion region[3] = {};
};
// Geometry and cover of an image; whether this form takes fewer instructions
// than the general adjoint on the image's pixels.
bool grid_plan(int nx, int ny, int cx, int cy, double cell, int prec, GridGeom* g, GridPlan* p);
size_t grid_row_bytes(const GridGeom& g);
size_t grid_slab_bytes(const GridGeom& g, int64_t rows);
size_t grid_partial_bytes(const GridGeom& g, int64_t n_chunks);
int64_t grid_chunk(const GridGeom& g, const GridPlan& p, int64_t rows, int n_cu);
// Adds `rows` rows in chunks of `chunk` to the partial sums (resume) or starts
// them.  y null: unit visibilities.
hipError_t launch_grid_slab(hipStream_t s, const GridGeom& g, const GridPlan& p, int64_t rows,
                            int64_t chunk, const double* u, const double* v, const double* w,
                            const void* y, int sign, bool resume, void* slab, double* partial);
// The FP32-compensated sums of all rows (chunk: the adjoint's).
hipError_t launch_image_f32c(hipStream_t s, const GridGeom& g, const GridPlan& plan, int64_t n_vis,
                             int64_t chunk, int n_cu, const double* u, const double* v,
                             const double* w, const void* y, int sign, double* partial);
hipError_t launch_grid_finish(hipStream_t s, const GridGeom& g, int prec, const double* partial,
                              int64_t n_chunks, int nx, int ny, int cx, int cy, int64_t n_vis,
                              double* img);

// Rows per chunk of the FP64 adjoint and of the gradients (ppl, cpl: groups of 64
// outputs per wave at most).
int64_t adjoint_cell_chunk(int64_t n_vis, int64_t n_pix, int ppl, int n_cu);
// Groups per wave of an adjoint, at most ppl.
int adjoint_cell_groups(int64_t n_vis, int64_t n_pix, int ppl, int n_cu);
int64_t grad_chunk(int64_t n_vis, int64_t n_comp, int cpl, int n_cu);
// Resident blocks per compute unit of the F32C adjoint.
int adjoint_f32c_blocks_per_cu(int ppl, int block);

// comp: packed components, {l, m, n - 1, I} at the start of every comp_stride
// doubles (4 for Comp, 8 for CompCell).  n_comp_dev (optional): the actual component count on the device, at most
// n_comp, which then only sizes the grid (see k_grad_cell).
hipError_t launch_grad(hipStream_t s, int cpl, int64_t chunk, int64_t n_vis, const double* u,
                       const double* v, const double* w, const void* y, const double* comp,
                       int comp_stride, int64_t n_comp, int sign, double alpha, double* partial,
                       double* d_flux, double* d_l, double* d_m,
                       const int* n_comp_dev = nullptr);

hipError_t launch_residual(hipStream_t s, int64_t n_vis, const void* obs, const void* model,
                           double inv_sigma2, void* resid, double* partial, double* chi2);

// Number of blocks launch_residual uses (its partial buffer holds that many doubles).
int residual_blocks(int64_t n_vis);

// ------------------------------------------------------------ batched --
// One prediction instance as the batched kernels read it.
struct BatchInst {
    const double* u;
    const double* v;
    const double* w;
    void* out;
    const double* l;      // direct: caller's components, packed into comp by the batched ingest
    const double* m;      // (an FP32-compensated instance: CompF records at its start)
    const double* flux;
    CompCell* comp;       // packed components; tree: its leaf sum (l null)
    int64_t n_vis;
    int n_comp;
    int prec;
    int is_tree;
    double sgn;
};

// A tile of rows [row0, row0 + nrows) of one instance; split: the FP64 kernel's
// waves share its rows' components.
struct WorkItem {
    int64_t row0;
    int inst;
    int nrows;
    int split;
    int unused;
};

hipError_t launch_batch_ingest(hipStream_t s, const BatchInst* inst, int n_inst, int max_comp,
                               int* status);
hipError_t launch_reset_counters(hipStream_t s, unsigned* counters, int n);
// Items of FP64 direct instances and of trees of either precision go through the
// first launch (a workgroup each), those of F32C direct instances through the
// second (persistent, batch_direct_f32c_blocks_per_cu() blocks of kBatchF32Block
// threads on each CU).
constexpr int kBatchRows = 2048, kBatchSplitRows = 256;
// Whether an instance's items share their rows' components: long lists (as
// direct_shape finds), and any list where whole rows would make less than four
// rounds of workgroups in all.
bool batch_split(int64_t total_rows, int64_t n_comp, int n_cu);
// Rows of its items: more than kBatchRows, and so fewer table fills, where that
// leaves 32 rounds of workgroups.
int batch_item_rows(int64_t total_rows, int64_t n_comp, int n_cu);
int batch_direct_f32c_blocks_per_cu();
constexpr int kBatchF32Vpl = 2, kBatchF32Block = 64;
hipError_t launch_batch_direct(hipStream_t s, const BatchInst* inst, const WorkItem* items,
                               unsigned n_items, int* status);
hipError_t launch_batch_direct_f32c(hipStream_t s, int grid, const BatchInst* inst,
                                    const WorkItem* items, unsigned n_items, unsigned* counter,
                                    int* status);

}  // namespace swv
