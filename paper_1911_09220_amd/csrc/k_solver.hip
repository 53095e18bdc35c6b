// Vector kernels of the preconditioned CG solver ("Scalable Linear Solvers":
// CG on the partially assembled operator; the paper notes that Krylov solvers
// run on the device because they are written with Vector operations, "GPU
// Acceleration").
//
// Each kernel is a grid of at most kCGBlocks x kCGThreads threads (one workgroup per
// compute unit) striding over the vectors.  Dot products: wave64 butterfly -> per-wave
// LDS -> one partial per workgroup, stored plainly; every workgroup of the next kernel
// of the iteration sums the (at most kCGBlocks) partials itself, in the same order, and
// so knows alpha, beta and convergence without another launch.  The first workgroup
// writes the scalars that the host or a later kernel reads.  Results do not depend on
// scheduling.  (A last-arriver reduction inside the kernel cost more than the vectors:
// its ticket and the device-wide fences, which write back the L2 of each die, took 10 us
// of a 14 us update on 4913 dofs, and the separate step-length kernel 12 us; with three
// kernels instead of four the iteration there went from 40 to 23 us, and at 1.3M dofs in
// 2D from 75 to 57 us.)
#include <algorithm>
#include <cmath>

#include "direction.hpp"
#include "internal.hpp"

namespace pafem {

namespace {

__device__ __forceinline__ bool state_done(const CGState* st) {
  return __hip_atomic_load(const_cast<int32_t*>(&st->done), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT) != 0;
}

// grid-stride loop, unrolled so each thread keeps several independent loads in flight
#define GRID_LOOP(i, n)                                                        \
  _Pragma("unroll 4")                                                          \
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < (n);    \
       i += int64_t(gridDim.x) * blockDim.x)

// Sum of a[0], a[stride], ... (n of them) over this thread's share; the block sum of it
// has a fixed order.
__device__ __forceinline__ double strided_share(const double* a, int n, int stride) {
  double v = 0.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += kCGThreads) v += a[size_t(i) * stride];
  return v;
}

// ---- one-workgroup kernels that turn partials into state --------------------
// (a solve's start and end; inside an iteration every workgroup of the next vector
// kernel sums the partials itself)

// p0 rz, p1 rr, p3 bb: start of a solve
__global__ void __launch_bounds__(kCGThreads)
    cg_start_finish_kernel(CGState* st, const double* partials, int nb, double rel_tol,
                           int32_t max_hist, double* hist, int flexible) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  double rr = strided_share(partials + kCGBlocks, nb, 1);
  double bb = strided_share(partials + 3 * kCGBlocks, nb, 1);
  block_sum2(rr, bb, scratch);
  double rz = flexible ? 0.0 : strided_share(partials, nb, 1);
  double ess = flexible ? 0.0 : strided_share(partials + 2 * kCGBlocks, nb, 1);
  block_sum2(rz, ess, scratch);
  if (threadIdx.x == 0) {
    // reference of the relative stop: ||b||^2, or ||r_0||^2 when b = 0 (the answer is
    // then x = 0 and the iteration reduces the initial residual; both 0: done)
    const double ref = bb > 0.0 ? bb : rr;
    st->rr = rr;
    st->bb = ref;
    st->tol2 = rel_tol * rel_tol * ref;
    if (!flexible) {
      st->rz = rz;
      st->ess = ess;
      st->alpha = st->beta = 0.0;
      st->res2 = 0.0;
    }
    if (max_hist >= 0) {  // negative: keep counting (restart inside a solve)
      st->iter = 0;
      st->max_hist = max_hist;
    }
    if (hist && st->max_hist > 0) hist[0] = ref > 0.0 ? sqrt(rr / ref) : 0.0;
    finish_done(st, rr <= st->tol2 ? 1 : 0);
  }
}

// p0 rz of the first preconditioned residual of flexible CG: must be > 0
__global__ void __launch_bounds__(kCGThreads)
    fcg_start_finish_kernel(CGState* st, const double* partials, int nb) {
  __shared__ double scratch[kCGThreads / kWave];
  if (state_done(st)) return;
  const double rz = block_sum(strided_share(partials, nb, 1), scratch);
  if (threadIdx.x == 0) {
    st->rz = rz;
    if (!(rz > 0.0) || !isfinite(rz)) finish_done(st, 3);
  }
}

__global__ void __launch_bounds__(kCGThreads)
    residual_finish_kernel(CGState* st, const double* partials, int nb) {
  __shared__ double scratch[kCGThreads / kWave];
  const double s = block_sum(strided_share(partials, nb, 1), scratch);
  if (threadIdx.x == 0) st->res2 = s;
}

// p0 rz, p1 rr of the (re)started inner PCG
__global__ void __launch_bounds__(kCGThreads)
    ir_start_finish_kernel(CGState* st, const double* partials, int nb, double inner_rel_tol) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  double rz = strided_share(partials, nb, 1), rr = strided_share(partials + kCGBlocks, nb, 1);
  block_sum2(rz, rr, scratch);
  const double ess = block_sum(strided_share(partials + 2 * kCGBlocks, nb, 1), scratch);
  if (threadIdx.x == 0) {
    st->rz = rz;
    st->ess = ess;
    st->rr = rr;
    st->bb = rr;
    st->tol2 = inner_rel_tol * inner_rel_tol * rr;
    st->iter = 0;
    st->alpha = st->beta = 0.0;
    finish_done(st, rr > 0.0 ? 0 : 1);
  }
}

// p0 rz, p1 rr, p2 z.q, p3 d.q after a residual replacement
__global__ void __launch_bounds__(kCGThreads)
    ir_replace_finish_kernel(CGState* st, const double* partials, int nb, double inner_rel_tol) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  double rz = strided_share(partials, nb, 1), rr = strided_share(partials + kCGBlocks, nb, 1);
  block_sum2(rz, rr, scratch);
  double zq = strided_share(partials + 2 * kCGBlocks, nb, 1);
  double dq = strided_share(partials + 3 * kCGBlocks, nb, 1);
  block_sum2(zq, dq, scratch);
  if (threadIdx.x == 0) {
    const double beta = -zq / dq;
    st->beta = beta;
    st->rz = rz;
    st->rr = rr;
    st->bb = rr;
    st->tol2 = inner_rel_tol * inner_rel_tol * rr;
    finish_done(st, (isfinite(beta) && rz > 0.0 && dq > 0.0) ? 0 : 2);
  }
}

// Element energies of an apply over more workgroups than a vector kernel's workgroups
// should each sum: workgroup b adds the entries of the 64-byte groups b, b + 256, ...
// into entry 8 b, which no other workgroup reads.
__global__ void __launch_bounds__(256) fold_kernel(double* __restrict__ e, int n) {
  __shared__ double scratch[256 / kWave];
  double v = 0.0;
#pragma unroll 4
  for (int64_t k = threadIdx.x / 8; k * (8 * kCGBlocks) < n; k += 32) {
    const int64_t i = k * (8 * kCGBlocks) + 8 * blockIdx.x + threadIdx.x % 8;
    if (i < n) v += e[i];
  }
  v = block_sum(v, scratch);
  if (threadIdx.x == 0) e[8 * blockIdx.x] = v;
}

// alpha = rz / (d . q) in every thread, d . q from the apply's element energies (epart)
// plus d_b^2 over the essential rows of a constrained operator (q_b = d_b there; pess,
// written with d): energy_share is the thread's part of it.  Returns false on breakdown
// (done = 2) in every workgroup.  st->rz is written only by direction kernels, rz_old only
// here.
__device__ __forceinline__ double energy_share(const EnergyParts& ep, const double* pess, int nb) {
  double s = strided_share(ep.e, ep.n, ep.stride);
  if (pess) s += strided_share(pess, nb, 1);
  return s;
}
__device__ __forceinline__ bool step_length(CGState* st, double share, double rz, double* scratch,
                                            const int& stopped, double& alpha) {
  const double pq = block_sum(share, scratch);
  if (stopped) return false;
  alpha = rz / pq;
  const bool ok = pq > 0.0 && isfinite(alpha);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->rz_old = rz;
    st->alpha = alpha;
    if (!ok) finish_done(st, 2);
  }
  return ok;
}

// Writes this block's partials of two sums (p0, p1).
__device__ __forceinline__ void put_partials2(double a, double b, double* p0, double* p1,
                                              double* scratch) {
  block_sum2(a, b, scratch);
  if (threadIdx.x == 0) {
    p0[blockIdx.x] = a;
    p1[blockIdx.x] = b;
  }
}

// r = b - q (q may be null: r = b), d = z = r / diag, x = 0 if zero_guess; partials
// rz, rr, bb and d_b^2 (p2); qi (may be null, may be q): the first apply's init of d
__global__ void __launch_bounds__(kCGThreads)
    cg_init_kernel(double* partials, const double* __restrict__ b, const double* q,
                   const double* __restrict__ diag, double* __restrict__ x,
                   double* __restrict__ r, double* __restrict__ d, double* qi,
                   const uint8_t* __restrict__ bmask, int zero_guess, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  double rz = 0.0, rr = 0.0, bb = 0.0, ess = 0.0;
  GRID_LOOP(i, n) {
    const double bi = b[i];
    const double ri = q ? bi - q[i] : bi;
    if (zero_guess) x[i] = 0.0;
    const double zi = diag ? ri / diag[i] : ri;
    r[i] = ri;
    d[i] = zi;
    const bool e = bmask && bmask[i];
    if (qi) qi[i] = e ? zi : 0.0;
    if (e) ess += zi * zi;
    rz += ri * zi;
    rr += ri * ri;
    bb += bi * bi;
  }
  put_partials2(rz, rr, partials, partials + kCGBlocks, scratch);
  put_partials2(ess, bb, partials + 2 * kCGBlocks, partials + 3 * kCGBlocks, scratch);
}

// The kernels of an iteration are chains of memory latencies on all but the largest
// vectors: flag, scalars and partials, then the vectors.  Each thread therefore issues the
// loads of its first kAhead entries before it waits for any of the scalars (pcg on 4913
// dofs: update 6.0 -> 5.3 us, direction 5.5 -> 5.1; at 1.3M dofs 14.3 -> 12.6 and 10.6 ->
// 9.0; FP32 refinement at 0.37M dofs 7.7 -> 6.5 and 6.7 -> 5.7).
constexpr int kAhead = 4;
#define AHEAD_LOOP(u, i, base, n)                                                       \
  _Pragma("unroll")                                                                     \
  for (int u = 0; u < kAhead; ++u)                                                      \
    if (const int64_t i = (base) + u * int64_t(gridDim.x) * kCGThreads; i < (n))
__device__ __forceinline__ int64_t first_entry() {
  return blockIdx.x * int64_t(kCGThreads) + threadIdx.x;
}
__device__ __forceinline__ int64_t entry_step() {
  return int64_t(gridDim.x) * kCGThreads * kAhead;
}

// x += alpha d; r -= alpha q; partials of rz and rr; q0 (null: none; may be q) = 0, the start
// of an apply that forms the next direction itself
__global__ void __launch_bounds__(kCGThreads)
    cg_update_kernel(CGState* st, EnergyParts ep, double* partials, int has_ess,
                     double* __restrict__ x, double* __restrict__ r,
                     const double* __restrict__ d, const double* q,
                     const double* __restrict__ diag, double* q0, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  __shared__ int stopped;
  read_done(st, &stopped);
  const double rz0 = st->rz;
  const double share =
      energy_share(ep, has_ess ? partials + 2 * kCGBlocks : nullptr, gridDim.x);
  double xv[kAhead], rv[kAhead], dv[kAhead], qv[kAhead], gv[kAhead];
  auto load = [&](int64_t base) {
    AHEAD_LOOP(u, i, base, n) {
      xv[u] = x[i];
      rv[u] = r[i];
      dv[u] = d[i];
      qv[u] = q[i];
      gv[u] = diag ? diag[i] : 1.0;
    }
  };
  load(first_entry());
  double alpha;
  if (!step_length(st, share, rz0, scratch, stopped, alpha)) return;
  double rz = 0.0, rr = 0.0;
  for (int64_t base = first_entry(); base < n; base += entry_step()) {
    if (base != first_entry()) load(base);
    AHEAD_LOOP(u, i, base, n) {
      x[i] = xv[u] + alpha * dv[u];
      if (q0) q0[i] = 0.0;
      const double ri = rv[u] - alpha * qv[u];
      r[i] = ri;
      const double zi = diag ? ri / gv[u] : ri;
      rz += ri * zi;
      rr += ri * ri;
    }
  }
  put_partials2(rz, rr, partials, partials + kCGBlocks, scratch);
}

// beta = rz / rz_old, state; d = r / diag + beta d; partials of d_b^2; q (null: the
// apply needs no init) = the next apply's init: d on essential dofs of a constrained
// operator (bmask non-null), 0 elsewhere
__global__ void __launch_bounds__(kCGThreads)
    cg_direction_kernel(CGState* st, double* partials, const double* __restrict__ r,
                        const double* __restrict__ diag, const double* d, double* dnew,
                        double* __restrict__ q, const uint8_t* __restrict__ bmask, double* hist,
                        int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  __shared__ int stopped;
  read_done(st, &stopped);
  const double rz_old = st->rz_old;
  double rz = strided_share(partials, gridDim.x, 1);
  double rr = strided_share(partials + kCGBlocks, gridDim.x, 1);
  double rv[kAhead], dv[kAhead], gv[kAhead];
  uint8_t ev[kAhead];
  auto load = [&](int64_t base) {
    AHEAD_LOOP(u, i, base, n) {
      rv[u] = r[i];
      dv[u] = d[i];
      gv[u] = diag ? diag[i] : 1.0;
      ev[u] = bmask ? bmask[i] : 0;
    }
  };
  load(first_entry());
  block_sum2(rz, rr, scratch);
  if (stopped) return;
  const double beta = rz / rz_old;
  if (close_update(st, rr, !isfinite(beta), hist)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) st->rz = rz;
    return;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->rz = rz;
    st->beta = beta;
  }
  double ess = 0.0;
  for (int64_t base = first_entry(); base < n; base += entry_step()) {
    if (base != first_entry()) load(base);
    AHEAD_LOOP(u, i, base, n) {
      const double zi = diag ? rv[u] / gv[u] : rv[u];
      const double di = zi + beta * dv[u];
      dnew[i] = di;
      if (q) q[i] = ev[u] ? di : 0.0;
      if (ev[u]) ess += di * di;
    }
  }
  if (bmask) {
    ess = block_sum(ess, scratch);
    if (threadIdx.x == 0) partials[2 * kCGBlocks + blockIdx.x] = ess;
  }
}

// ---- flexible CG (variable preconditioner) ----
// r = b - q (q may be null), x = 0 if zero_guess; partials rr, bb
__global__ void __launch_bounds__(kCGThreads)
    fcg_init_kernel(double* partials, const double* __restrict__ b, const double* __restrict__ q,
                    double* __restrict__ x, double* __restrict__ r, int zero_guess, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  double rr = 0.0, bb = 0.0;
  GRID_LOOP(i, n) {
    const double bi = b[i];
    const double ri = q ? bi - q[i] : bi;
    if (zero_guess) x[i] = 0.0;
    r[i] = ri;
    rr += ri * ri;
    bb += bi * bi;
  }
  put_partials2(rr, bb, partials + kCGBlocks, partials + 3 * kCGBlocks, scratch);
}

// p = z; partials of r . z and p_b^2; q = the apply's init of p (null: none)
__global__ void __launch_bounds__(kCGThreads)
    fcg_start_kernel(const CGState* st, double* partials, const double* __restrict__ r,
                     const double* __restrict__ z, double* __restrict__ p,
                     double* __restrict__ q, const uint8_t* __restrict__ bmask, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  if (state_done(st)) return;
  double rz = 0.0, ess = 0.0;
  GRID_LOOP(i, n) {
    const double zi = z[i];
    p[i] = zi;
    const bool e = bmask && bmask[i];
    if (q) q[i] = e ? zi : 0.0;
    if (e) ess += zi * zi;
    rz += r[i] * zi;
  }
  put_partials2(rz, ess, partials, partials + 2 * kCGBlocks, scratch);
}

// x += alpha p; r -= alpha q; zj = r / diag (r on essential dofs: the Jacobi part of
// the next preconditioned residual); partials of rr
__global__ void __launch_bounds__(kCGThreads)
    fcg_update_kernel(CGState* st, EnergyParts ep, double* partials, double* __restrict__ x,
                      double* __restrict__ r, const double* __restrict__ p,
                      const double* __restrict__ q, const double* __restrict__ diag,
                      const uint8_t* __restrict__ bmask, double* __restrict__ zj, int64_t n) {
  __shared__ double scratch[kCGThreads / kWave];
  __shared__ int stopped;
  read_done(st, &stopped);
  const double rz0 = st->rz;
  const double share = energy_share(ep, bmask ? partials + 2 * kCGBlocks : nullptr, gridDim.x);
  double alpha;
  if (!step_length(st, share, rz0, scratch, stopped, alpha)) return;
  double rr = 0.0;
  GRID_LOOP(i, n) {
    x[i] += alpha * p[i];
    const double ri = r[i] - alpha * q[i];
    r[i] = ri;
    zj[i] = (bmask && bmask[i]) ? ri : ri / diag[i];
    rr += ri * ri;
  }
  rr = block_sum(rr, scratch);
  if (threadIdx.x == 0) partials[kCGBlocks + blockIdx.x] = rr;
}

// state after the update; partials of r . z (p0) and r . z_old (p3)
__global__ void __launch_bounds__(kCGThreads)
    fcg_beta_kernel(CGState* st, double* partials, const double* __restrict__ r,
                    const double* __restrict__ z, const double* __restrict__ zold, double* hist,
                    int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  __shared__ int stopped;
  read_done(st, &stopped);
  const double rr = block_sum(strided_share(partials + kCGBlocks, gridDim.x, 1), scratch);
  if (stopped) return;
  if (close_update(st, rr, false, hist)) return;
  double rz = 0.0, rzo = 0.0;
  GRID_LOOP(i, n) {
    const double ri = r[i];
    rz += ri * z[i];
    rzo += ri * zold[i];
  }
  put_partials2(rz, rzo, partials, partials + 3 * kCGBlocks, scratch);
}

// beta = r.(z - z_old) / rz_old (Polak-Ribiere; r.z > 0 else done = 3); p = z + beta p;
// q = the next apply's init of p (null: none)
__global__ void __launch_bounds__(kCGThreads)
    fcg_direction_kernel(CGState* st, double* partials, const double* __restrict__ z,
                         double* __restrict__ p, double* __restrict__ q,
                         const uint8_t* __restrict__ bmask, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  __shared__ int stopped;
  read_done(st, &stopped);
  double rz = strided_share(partials, gridDim.x, 1);
  double rzo = strided_share(partials + 3 * kCGBlocks, gridDim.x, 1);
  block_sum2(rz, rzo, scratch);
  if (stopped) return;
  const double beta = (rz - rzo) / st->rz_old;
  const bool ok = rz > 0.0 && isfinite(beta);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->beta = beta;
    st->rz = rz;
    if (!ok) finish_done(st, 3);
  }
  if (!ok) return;
  double ess = 0.0;
  GRID_LOOP(i, n) {
    const double pi = z[i] + beta * p[i];
    p[i] = pi;
    const bool e = bmask && bmask[i];
    if (q) q[i] = e ? pi : 0.0;
    if (e) ess += pi * pi;
  }
  if (bmask) {
    ess = block_sum(ess, scratch);
    if (threadIdx.x == 0) partials[2 * kCGBlocks + blockIdx.x] = ess;
  }
}

__global__ void __launch_bounds__(kCGThreads)
    residual_kernel(double* partials, const double* __restrict__ b, const double* __restrict__ q,
                    double* __restrict__ r, int64_t n) {
  __shared__ double scratch[kCGThreads / kWave];
  double s = 0.0;
  GRID_LOOP(i, n) {
    const double v = b[i] - q[i];
    if (r) r[i] = v;
    s += v * v;
  }
  s = block_sum(s, scratch);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// ---- inner PCG of iterative refinement --------------------------------------
// The inner solve of A_lo d = r / s keeps its residual r, the preconditioned
// residual z, all dot products and the solution x in FP64 (x += s alpha d
// directly, so the FP64 residual b - A x that replaces r carries no rounding of
// an intermediate correction); only what the reduced-precision apply reads and
// writes is FP32: the direction d and its image q = A_lo d.  dinv is the Jacobi
// preconditioner 1/diag rounded to FP32 (a preconditioner, not part of the
// answer); null for none.  Essential rows: q_b = d_b for a constrained operator.

// r *= inv_s (r holds the FP64 residual), d = z, q = apply init of d; partials of rz,
// rr and d_b^2
__global__ void __launch_bounds__(kCGThreads)
    ir_start_kernel(double* partials, double* __restrict__ r, double inv_s,
                    const float* __restrict__ dinv, float* __restrict__ d, float* __restrict__ q,
                    const uint8_t* __restrict__ ess, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  double rz = 0.0, rr = 0.0, de = 0.0;
  GRID_LOOP(i, n) {
    const double ri = r[i] * inv_s;
    r[i] = ri;
    const double zi = dinv ? ri * double(dinv[i]) : ri;
    const float di = float(zi);
    d[i] = di;
    const bool e = ess && ess[i];
    q[i] = e ? di : 0.0f;
    if (e) de += double(di) * double(di);
    rz += ri * zi;
    rr += ri * ri;
  }
  put_partials2(rz, rr, partials, partials + kCGBlocks, scratch);
  de = block_sum(de, scratch);
  if (threadIdx.x == 0) partials[2 * kCGBlocks + blockIdx.x] = de;
}

// x += (s alpha) d; r -= alpha q (FP64); partials of rz and rr
__global__ void __launch_bounds__(kCGThreads)
    ir_update_kernel(CGState* st, EnergyParts ep, double* partials, int has_ess,
                     double* __restrict__ x, double s, double* __restrict__ r,
                     const float* __restrict__ d, const float* __restrict__ q,
                     const float* __restrict__ dinv, float* __restrict__ q0, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  __shared__ int stopped;
  read_done(st, &stopped);
  const double rz0 = st->rz;
  const double share =
      energy_share(ep, has_ess ? partials + 2 * kCGBlocks : nullptr, gridDim.x);
  double xv[kAhead], rv[kAhead];
  float dv[kAhead], qv[kAhead], gv[kAhead];
  auto load = [&](int64_t base) {
    AHEAD_LOOP(u, i, base, n) {
      xv[u] = x[i];
      rv[u] = r[i];
      dv[u] = d[i];
      qv[u] = q[i];
      gv[u] = dinv ? dinv[i] : 1.0f;
    }
  };
  load(first_entry());
  double alpha;
  if (!step_length(st, share, rz0, scratch, stopped, alpha)) return;
  const double xstep = s * alpha;
  double rz = 0.0, rr = 0.0;
  for (int64_t base = first_entry(); base < n; base += entry_step()) {
    if (base != first_entry()) load(base);
    AHEAD_LOOP(u, i, base, n) {
      x[i] = xv[u] + xstep * double(dv[u]);
      if (q0) q0[i] = 0.0f;
      const double ri = rv[u] - alpha * double(qv[u]);
      r[i] = ri;
      const double zi = ri * double(gv[u]);
      rz += ri * zi;
      rr += ri * ri;
    }
  }
  put_partials2(rz, rr, partials, partials + kCGBlocks, scratch);
}

// d = z + beta d (stored FP32), q = apply init of the new d; partials of d_b^2.
// beta and the state as in cg_direction_kernel, or (replaced) the beta that the
// residual replacement left in the state.
__global__ void __launch_bounds__(kCGThreads)
    ir_direction_kernel(CGState* st, double* partials, int replaced, const double* __restrict__ r,
                        const float* __restrict__ dinv, const float* d, float* dnew,
                        float* __restrict__ q, const uint8_t* __restrict__ ess, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  __shared__ int stopped;
  read_done(st, &stopped);
  const double rz_old = st->rz_old;
  double beta = st->beta;
  double rz = strided_share(partials, gridDim.x, 1);
  double rr = strided_share(partials + kCGBlocks, gridDim.x, 1);
  double rv[kAhead];
  float dv[kAhead], gv[kAhead];
  uint8_t ev[kAhead];
  auto load = [&](int64_t base) {
    AHEAD_LOOP(u, i, base, n) {
      rv[u] = r[i];
      dv[u] = d[i];
      gv[u] = dinv ? dinv[i] : 1.0f;
      ev[u] = ess ? ess[i] : 0;
    }
  };
  load(first_entry());
  block_sum2(rz, rr, scratch);
  if (stopped) return;
  if (!replaced) {
    beta = rz / rz_old;
    const bool stop = close_update(st, rr, !isfinite(beta), nullptr);
    if (blockIdx.x == 0 && threadIdx.x == 0) st->rz = rz;
    if (stop) return;
  }
  double de = 0.0;
  for (int64_t base = first_entry(); base < n; base += entry_step()) {
    if (base != first_entry()) load(base);
    AHEAD_LOOP(u, i, base, n) {
      const float di = float(rv[u] * double(gv[u]) + beta * double(dv[u]));
      dnew[i] = di;
      q[i] = ev[u] ? di : 0.0f;
      if (ev[u]) de += double(di) * double(di);
    }
  }
  if (ess) {
    de = block_sum(de, scratch);
    if (threadIdx.x == 0) partials[2 * kCGBlocks + blockIdx.x] = de;
  }
}

// Residual replacement: r holds the FP64 residual b - A_hi x; scale it by 1/s_new
// and continue the recurrence with the kept direction d.  The next
// direction d' = z + beta d is made A_lo-conjugate to d using q = A_lo d of the
// last step: beta = -(z . q) / (d . q).  Without rounding and operator mismatch this
// is the usual beta in the new scaling (times s_old / s_new for the kept direction);
// with a replaced residual it keeps at least the last direction conjugate.
__global__ void __launch_bounds__(kCGThreads)
    ir_replace_kernel(double* partials, double* __restrict__ r, double inv_s_new,
                      const float* __restrict__ dinv, const float* __restrict__ d,
                      const float* __restrict__ q, int64_t n) {
  __shared__ double scratch[2 * kCGThreads / kWave];
  double rz = 0.0, rr = 0.0, zq = 0.0, dq = 0.0;
  GRID_LOOP(i, n) {
    const double ri = r[i] * inv_s_new;
    r[i] = ri;
    const double zi = dinv ? ri * double(dinv[i]) : ri;
    const double qi = double(q[i]);
    rz += ri * zi;
    rr += ri * ri;
    zq += zi * qi;
    dq += double(d[i]) * qi;
  }
  put_partials2(rz, rr, partials, partials + kCGBlocks, scratch);
  put_partials2(zq, dq, partials + 2 * kCGBlocks, partials + 3 * kCGBlocks, scratch);
}

// dinv = 1 / diag rounded to FP32
__global__ void __launch_bounds__(kCGThreads)
    ir_dinv_kernel(const double* __restrict__ diag, float* __restrict__ dinv, int64_t n) {
  GRID_LOOP(i, n) dinv[i] = float(1.0 / diag[i]);
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
  const uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u)  // inf or nan
    return uint16_t((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  const uint32_t rounding = 0x7fffu + ((u >> 16) & 1u);
  return uint16_t((u + rounding) >> 16);
}

__global__ void __launch_bounds__(kCGThreads)
    convert_kernel(const double* __restrict__ src, void* __restrict__ dst, int dtype, int64_t n) {
  GRID_LOOP(i, n) {
    const float f = float(src[i]);
    if (dtype == PAFEM_F32)
      static_cast<float*>(dst)[i] = f;
    else
      static_cast<uint16_t*>(dst)[i] = f32_to_bf16_bits(f);
  }
}

void check_launch(const char* what) {
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) throw Error(PAFEM_EHIP, std::string(what) + ": " + hipGetErrorString(err));
}

int vec_grid(int64_t n) {
  int64_t g = (n + kCGThreads - 1) / kCGThreads;
  return int(g < 1 ? 1 : (g > 65536 ? 65536 : g));
}

// workgroups of a vector kernel, and so partials of each of its sums: one element per
// thread until every compute unit has a workgroup (a fixed grid would leave most of its
// workgroups empty on small vectors, where their start and their partials are the time)
int cg_blocks(int64_t n) {
  return int(std::min<int64_t>(kCGBlocks, std::max<int64_t>(1, (n + kCGThreads - 1) / kCGThreads)));
}

}  // namespace

Direction make_direction(CGState* st, const double* partials, double* hist, const double* r,
                         const void* scale, const void* dold, void* dnew, int64_t n) {
  return {st, partials, hist, r, scale, dold, dnew, cg_blocks(n)};
}

namespace {

#define CG_LAUNCH(kernel, n, s, ...)                                                          \
  hipLaunchKernelGGL(kernel, dim3(cg_blocks(n)), dim3(kCGThreads), 0, s, __VA_ARGS__);        \
  check_launch(#kernel)
#define CG_FINISH(kernel, s, ...)                                                             \
  hipLaunchKernelGGL(kernel, dim3(1), dim3(kCGThreads), 0, s, __VA_ARGS__);                   \
  check_launch(#kernel)

EnergyParts energy_parts(double* epart, int nepart, hipStream_t s) {
  if (fold_kernels(nepart) == 0) return {epart, nepart, 1};
  hipLaunchKernelGGL(fold_kernel, dim3(kCGBlocks), dim3(256), 0, s, epart, nepart);
  check_launch("fold_kernel");
  return {epart, kCGBlocks, 8};
}

}  // namespace

void launch_cg_init(CGState* st, double* partials, const double* b, const double* q,
                    const double* diag, double* x, double* r, double* d, double* qi,
                    const uint8_t* bmask, int zero_guess, double rel_tol, int32_t max_hist,
                    double* hist, int64_t n, hipStream_t s) {
  CG_LAUNCH(cg_init_kernel, n, s, partials, b, q, diag, x, r, d, qi, bmask, zero_guess, n);
  CG_FINISH(cg_start_finish_kernel, s, st, partials, cg_blocks(n), rel_tol, max_hist, hist, 0);
}

void launch_cg_update(CGState* st, double* partials, double* epart, int nepart, bool has_ess,
                      double* x, double* r, const double* d, const double* q, const double* diag,
                      double* q0, int64_t n, hipStream_t s) {
  const EnergyParts ep = energy_parts(epart, nepart, s);
  CG_LAUNCH(cg_update_kernel, n, s, st, ep, partials, int(has_ess), x, r, d, q, diag, q0, n);
}

void launch_cg_direction(CGState* st, double* partials, const double* r, const double* diag,
                         const double* d, double* dnew, double* q, const uint8_t* bmask,
                         double* hist, int64_t n, hipStream_t s) {
  CG_LAUNCH(cg_direction_kernel, n, s, st, partials, r, diag, d, dnew, q, bmask, hist, n);
}

void launch_fcg_init(CGState* st, double* partials, const double* b, const double* q, double* x,
                     double* r, int zero_guess, double rel_tol, int32_t max_hist, double* hist,
                     int64_t n, hipStream_t s) {
  CG_LAUNCH(fcg_init_kernel, n, s, partials, b, q, x, r, zero_guess, n);
  CG_FINISH(cg_start_finish_kernel, s, st, partials, cg_blocks(n), rel_tol, max_hist, hist, 1);
}
void launch_fcg_start(CGState* st, double* partials, const double* r, const double* z, double* p,
                      double* q, const uint8_t* bmask, int64_t n, hipStream_t s) {
  CG_LAUNCH(fcg_start_kernel, n, s, st, partials, r, z, p, q, bmask, n);
  CG_FINISH(fcg_start_finish_kernel, s, st, partials, cg_blocks(n));
}
void launch_fcg_update(CGState* st, double* partials, double* epart, int nepart, double* x,
                       double* r, const double* p, const double* q, const double* diag,
                       const uint8_t* bmask, double* zj, int64_t n, hipStream_t s) {
  const EnergyParts ep = energy_parts(epart, nepart, s);
  CG_LAUNCH(fcg_update_kernel, n, s, st, ep, partials, x, r, p, q, diag, bmask, zj, n);
}
void launch_fcg_beta(CGState* st, double* partials, const double* r, const double* z,
                     const double* zold, double* hist, int64_t n, hipStream_t s) {
  CG_LAUNCH(fcg_beta_kernel, n, s, st, partials, r, z, zold, hist, n);
}
void launch_fcg_direction(CGState* st, double* partials, const double* z, double* p, double* q,
                          const uint8_t* bmask, int64_t n, hipStream_t s) {
  CG_LAUNCH(fcg_direction_kernel, n, s, st, partials, z, p, q, bmask, n);
}

void launch_residual(CGState* st, double* partials, const double* b, const double* q, double* r,
                     int64_t n, hipStream_t s) {
  CG_LAUNCH(residual_kernel, n, s, partials, b, q, r, n);
  CG_FINISH(residual_finish_kernel, s, st, partials, cg_blocks(n));
}

void launch_ir_start(CGState* st, double* partials, double* r, double s, const float* dinv,
                     float* d, float* q, const uint8_t* ess, double inner_rel_tol, int64_t n,
                     hipStream_t stream) {
  CG_LAUNCH(ir_start_kernel, n, stream, partials, r, 1.0 / s, dinv, d, q, ess, n);
  CG_FINISH(ir_start_finish_kernel, stream, st, partials, cg_blocks(n), inner_rel_tol);
}

void launch_ir_update(CGState* st, double* partials, double* epart, int nepart, bool has_ess,
                      double* x, double s, double* r, const float* d, const float* q,
                      const float* dinv, float* q0, int64_t n, hipStream_t stream) {
  const EnergyParts ep = energy_parts(epart, nepart, stream);
  CG_LAUNCH(ir_update_kernel, n, stream, st, ep, partials, int(has_ess), x, s, r, d, q, dinv, q0,
            n);
}

void launch_ir_direction(CGState* st, double* partials, bool replaced, const double* r,
                         const float* dinv, const float* d, float* dnew, float* q,
                         const uint8_t* ess, int64_t n, hipStream_t stream) {
  CG_LAUNCH(ir_direction_kernel, n, stream, st, partials, int(replaced), r, dinv, d, dnew, q, ess,
            n);
}

void launch_ir_replace(CGState* st, double* partials, double* r, double s_new, const float* dinv,
                       const float* d, const float* q, double inner_rel_tol, int64_t n,
                       hipStream_t stream) {
  CG_LAUNCH(ir_replace_kernel, n, stream, partials, r, 1.0 / s_new, dinv, d, q, n);
  CG_FINISH(ir_replace_finish_kernel, stream, st, partials, cg_blocks(n), inner_rel_tol);
}

void launch_ir_dinv(const double* diag, float* dinv, int64_t n, hipStream_t stream) {
  hipLaunchKernelGGL(ir_dinv_kernel, dim3(vec_grid(n)), dim3(kCGThreads), 0, stream, diag, dinv,
                     n);
  check_launch("ir_dinv");
}

void launch_convert(const double* src, void* dst, int dtype, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(convert_kernel, dim3(vec_grid(n)), dim3(kCGThreads), 0, s, src, dst, dtype,
                     n);
  check_launch("convert");
}

}  // namespace pafem
