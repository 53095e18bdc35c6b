// The CG direction step inside an operator action: what the fused apply kernels
// (k_apply.hip, k_2d.hip) need of the solver, and the parts of it that they share with the
// solver's own kernels (k_solver.hip).
#pragma once

#include "device.hpp"
#include "solver.hpp"

namespace pafem {

__device__ __forceinline__ void finish_done(CGState* st, int done) {
  __hip_atomic_store(&st->done, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// done as this workgroup saw it, into LDS: valid for all threads after the next barrier, and
// so the same for all of them.  The first workgroup of a launch may store done while others
// start: read by every wave for itself, some waves of such a workgroup would leave and the rest
// sum LDS slots that were never written.
__device__ __forceinline__ void read_done(const CGState* st, int* stopped) {
  if (threadIdx.x == 0)
    *stopped = __hip_atomic_load(const_cast<int32_t*>(&st->done), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
}

// State after an update: convergence on rr, history, iteration count.  Same decision
// in every workgroup that has not seen done yet, written by the first; returns true when the
// iteration stops.
__device__ __forceinline__ bool close_update(CGState* st, double rr, bool broken, double* hist) {
  const int done = (!isfinite(rr) || broken) ? 2 : rr <= st->tol2 ? 1 : 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->rr = rr;
    const int it = st->iter + 1;
    st->iter = it;
    if (hist && it < st->max_hist) hist[it] = sqrt(rr / st->bb);
    if (done) finish_done(st, done);
  }
  return done != 0;
}

// beta = rz / rz_old from the last update's partials in every thread, and the state as
// the direction kernels leave it; false when the iteration has stopped.  `scratch`: 2 doubles
// per wave.  Contains __syncthreads().
__device__ __forceinline__ bool direction_beta(const Direction& d, double* scratch, double& beta) {
  __shared__ int stopped;
  read_done(d.st, &stopped);
  const double rz_old = d.st->rz_old;
  double rz = 0.0, rr = 0.0;
  for (int i = threadIdx.x; i < d.nb; i += blockDim.x) {
    rz += d.partials[i];
    rr += d.partials[kCGBlocks + i];
  }
  block_sum2(rz, rr, scratch);
  if (stopped) return false;
  beta = rz / rz_old;
  const bool stop = close_update(d.st, rr, !isfinite(beta), d.hist);
  if (blockIdx.x == 0 && threadIdx.x == 0) d.st->rz = rz;
  return !stop;
}

// One entry of the new direction.  Several tiles may hold the dof: all store the same value.
__device__ __forceinline__ double direction_entry(const Direction& d, double beta, int g) {
  const double* diag = static_cast<const double*>(d.scale);
  const double r = d.r[g];
  const double v = (diag ? r / diag[g] : r) + beta * static_cast<const double*>(d.dold)[g];
  static_cast<double*>(d.dnew)[g] = v;
  return v;
}
// the inner PCG of refinement: FP32 direction and inverse diagonal, the rest in FP64
__device__ __forceinline__ float direction_entry_f32(const Direction& d, double beta, int g) {
  const float* dinv = static_cast<const float*>(d.scale);
  const double r = d.r[g];
  const float v = float((dinv ? r * double(dinv[g]) : r) +
                        beta * double(static_cast<const float*>(d.dold)[g]));
  static_cast<float*>(d.dnew)[g] = v;
  return v;
}

}  // namespace pafem
