// Device-resident view of a packed model, passed by value to the kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "forest_plan.hpp"

namespace forest_impl {

// Lays a workspace out in `bytes` bytes at `base` (256-byte aligned): the rank tiles first, sized
// for `tiles` row tiles of the model, the partial sums in the rest.
Workspace carve_workspace(const DevModel &m, void *base, size_t bytes, int64_t tiles);

// Bytes of a workspace that never limits a split launch of the model.
size_t full_workspace_bytes(int rank_regs, int n_outputs);

// Enqueues one pass over `n_rows` rows on `stream`.  `scores` / `labels` / `leaf_out` may be
// null (that part is not written).  `ws` is the workspace a small batch may use (null: the trees
// are never cut into shares).  With `must_fit`, a small batch whose split launch does not fit
// `ws` is refused with hipErrorMemoryAllocation instead of being run unsplit.  Returns the launch
// error, if any.
hipError_t launch_predict(const DevModel &m, const Workspace *ws, bool must_fit, const float *X, int64_t n_rows,
                          float *scores, int32_t *labels, int32_t *leaf_out, hipStream_t stream);

// The calling device's copy of the library's static scratch array (set up by init_kernels), and
// its size in bytes; null before init_kernels has run on the device.
void *static_scratch(int device);
size_t static_scratch_bytes();

// Register-resident family (forest_kernels_reg.hip).
hipError_t init_reg_kernels(size_t lds_limit);
hipError_t launch_reg(const DevModel &m, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                      int32_t *leaf_out, hipStream_t stream);

// Rank family (forest_kernels_rank.hip).
hipError_t init_rank_kernels(size_t lds_limit);
hipError_t launch_rank(const DevModel &m, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                       int32_t *leaf_out, hipStream_t stream);

// LDS-resident rank family (forest_kernels_ranklds.hip).
hipError_t init_ranklds_kernels(size_t lds_limit);
hipError_t launch_ranklds(const DevModel &m, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                          int32_t *leaf_out, size_t lds_limit, hipStream_t stream);

// Register-bank kernel of the LDS rank family (forest_kernels_rankbank.hip).
hipError_t init_rankbank_kernels(size_t lds_limit);
hipError_t launch_rankbank(const DevModel &m, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                           int32_t *leaf_out, size_t lds_limit, hipStream_t stream);

// Walk kernels (forest_kernels_walk.hip).  t: the workgroups of the rows at hand, of which m.full_workgroups holds the first number.
hipError_t init_walk_kernels(size_t lds_limit);
hipError_t launch_walk(const DevModel &m, int groups, const TailPlan &t, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                       int32_t *leaf_out, hipStream_t stream);

// Deep walk kernels (forest_kernels_deep.hip).
hipError_t init_deep_kernels(size_t lds_limit);
hipError_t launch_deep(const DevModel &m, int groups, const TailPlan &t, const float *X, int64_t n_rows, float *scores, int32_t *labels,
                       int32_t *leaf_out, hipStream_t stream);

hipError_t launch_deep_tiles(const DevModel &m, const float *X, int64_t n_rows, float *scores, int32_t *labels, hipStream_t stream);

// One lane per (row, tree) (forest_kernels_split.hip).
hipError_t launch_point(const DevModel &m, const float *X, int64_t n_rows, float *scores, int32_t *labels, int32_t *leaf_out,
                        hipStream_t stream);

// Sums the partial sums of a split launch over the splits and finishes every row.
hipError_t launch_reduce_splits(const DevModel &m, int64_t n_rows, float *scores, int32_t *labels,
                                hipStream_t stream);

// Threshold ranks of every 128-row tile of the batch into m.rank_tiles (rank families).
hipError_t launch_rank_tiles(const DevModel &m, const float *X, int64_t n_rows, hipStream_t stream);

// Whether the kernels' LDS working set for this model fits a compute unit (host-only check).
bool model_fits(const PackedModel &m);

// One-time per-process kernel attribute setup (dynamic LDS limits).
hipError_t init_kernels();

}  // namespace forest_impl
