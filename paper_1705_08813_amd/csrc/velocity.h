// Velocity residual: what the kernels of cells without enrichment and the
// general ones share.
#pragma once

#include "kern_common.h"

namespace dgwm {

// One mesh of a batched launch.
struct VelBatchItem {
  MeshDev M;
  const void* u;
  void* r;
  int layer_lo, nlayers;
  int ncells;
};

// Item that owns this block (prefix[i]: first block of item i), uniform over
// the wavefront.
__device__ __forceinline__ int batch_item(const int64_t* __restrict__ prefix, int nitems) {
  const int64_t b = blockIdx.x;
  int lo = 0, hi = nitems;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (prefix[mid] <= b) lo = mid; else hi = mid;
  }
  return __builtin_amdgcn_readfirstlane(lo);
}

// r = R(u) (viscous: with the viscous terms) on the layers [lo, lo + nl) of
// cells without enrichment; enriched neighbours with constant weights (l = 0)
template <typename T>
int launch_residual_regular(const dg_mesh* m, const T* u, T* r, int lo, int nl, bool viscous, hipStream_t s);
// the same over the items of one (k + 1, n_q): prefix counts workgroups of
// residual_cells_per_block cells
template <typename T>
int launch_residual_regular_batched(int np, int nq, const VelBatchItem* items, const int64_t* prefix, int n,
                                    int64_t blocks, hipStream_t s);
int residual_cells_per_block(int np);

}  // namespace dgwm
