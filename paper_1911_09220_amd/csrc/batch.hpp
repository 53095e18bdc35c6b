// Batched multi-right-hand-side apply over many meshes: device descriptors and
// launchers (k_batch.hip), used by the host batch object (batch.cpp).
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "internal.hpp"

namespace pafem {

// One mesh of a batch, as the kernels see it.
struct BatchMesh {
  const int32_t* gmap;   // device-order element->dof map, ~g on essential dofs
  const uint8_t* bmask;  // essential-dof mask
  const void* qdata;     // tile-interleaved quadrature data
  const void* x;         // [ndofs][nrhs]
  void* y;               // [ndofs][nrhs]
  int32_t ne, ndofs;
  int32_t tile_begin;    // first tile of this mesh among its order's
  int32_t constrained;
};

// candidates 0..4: vector-unit tiles (k_batch.hip); 5: FP64 matrix cores, one element x
// 16 right-hand sides per workgroup (k_batch_mfma.hip), orders 1..4
constexpr int kBatchCandidates = 6;
constexpr int kBatchMfmaCandidate = 5;
int batch_tile_elems(int cand);
int batch_tile_rhs(int cand);
// Groups of right-hand sides in one launch, one workgroup of `threads` for each tile and group:
// all of them, or as even a share as keeps the launch under the 2^32 threads that a grid's
// first dimension may have (1e6 elements at p = 1 reach them at 478 right-hand sides)
inline int batch_launch_groups(int64_t tiles, int threads, int groups) {
  const int64_t most = int64_t(0xffffffff) / (tiles * threads);
  if (most < 1) return 1;  // tiles alone are too many: the launch is refused
  const int64_t launches = (groups + most - 1) / most;
  return int((groups + launches - 1) / launches);
}
// Launches the multi-rhs apply of one order group; false if the (order,
// candidate, dtype) combination is not built.
// tabB: the order's 1D B table followed by its G table, in the vector dtype
bool launch_batch_apply(int p, int cand, int vdtype, int qdtype, int kind,
                        const BatchMesh* meshes, int nmesh, int64_t ntiles, const void* tabB,
                        int nrhs, hipStream_t st);
void launch_batch_init(int vdtype, const BatchMesh* meshes, int nmesh, int nrhs, hipStream_t st);
// the matrix-core variant (FP64, orders 1..4, nrhs a multiple of 16); false otherwise
bool launch_batch_apply_mfma(int p, int kind, const BatchMesh* meshes, int nmesh, int ntiles,
                             const double* tabB, int nrhs, hipStream_t st);

}  // namespace pafem
