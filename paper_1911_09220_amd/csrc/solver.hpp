// Device-resident state of the preconditioned CG solver and its launchers.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

namespace pafem {

// Lives at the start of the solver workspace.  Every scalar of the iteration
// stays on the device; the host only reads `done`/`iter` now and then.
struct CGState {
  double rz;     // r . z of the current residual
  double alpha;  // step length of the current iteration
  double beta;   // direction update factor
  double rr;     // r . r
  double bb;     // b . b
  double tol2;   // rel_tol^2 * b . b
  double res2;   // ||b - A x||^2 computed at exit
  double rz_old; // rz at the last update (the denominator of beta)
  double ess;    // sum of d_b^2 over the essential rows at the start
  int32_t iter;  // completed iterations
  int32_t done;  // 0 running, 1 converged, 2 breakdown, 3 preconditioner not positive
  int32_t max_hist;
  int32_t pad1;
};

constexpr int kCGBlocks = 256;  // most workgroups of a vector kernel = partials per sum
constexpr int kCGThreads = 1024;
// Partials of one solver: kPartials arrays of kCGBlocks doubles.  p0: r.z; p1: r.r; p2: d_b^2
// over the essential rows, written with the direction and read by the next update; p3:
// b.b at the start, r.z_old in flexible CG.  No kernel writes an array that it reads.
constexpr int kPartials = 4;

// The element energies of an apply (one per workgroup) as the update kernels read them:
// n entries, stride apart.  Up to kFoldAbove of them every workgroup of the update sums
// them all itself; a larger apply's are folded to kCGBlocks first, in place.  The fold's
// launch costs 1-3 us an iteration up to 17562 of them (p = 1, 40^3 elements: 38.8 us
// folded, 35.8 direct), nothing at 31598, and gains 4 of 523 us at 74899 (p = 1, 128^3).
struct EnergyParts {
  const double* e;
  int n, stride;
};
constexpr int kFoldAbove = 32768;
inline int fold_kernels(int nepart) { return nepart > kFoldAbove ? 1 : 0; }

// The direction step of an iteration as part of the apply that follows it (FP64 and FP32
// diffusion): the kernel sums rz and rr of the last update (partials, nb of each), decides
// convergence, and forms d = z + beta d_old where it gathers its input, stored to dnew.
// scale: the FP64 diagonal (z = r / diag) or the FP32 inverse diagonal (z = r dinv); null:
// z = r.  Only where d is 0 on the essential rows: they are 0 in every later iteration then,
// and need neither y's start nor their part of d . q.
struct Direction {
  CGState* st;
  const double* partials;
  double* hist;
  const double* r;
  const void* scale;
  const void* dold;
  void* dnew;
  int nb;
};
Direction make_direction(CGState* st, const double* partials, double* hist, const double* r,
                         const void* scale, const void* dold, void* dnew, int64_t n);

// Dot products always accumulate in double.  Every apply between two kernels below
// passes its element energies as epart (nepart of them, overwritten).  q / qi arguments
// receive the next apply's init (d on the essential dofs given by bmask, 0 elsewhere;
// bmask null: 0 everywhere); null: the apply needs none.
//
// r = b - q (q may be null; qi may be q); x = 0 if zero_guess; d = z = r / diag; sets
// the whole state, hist[0]; hist holds max_hist entries
void launch_cg_init(CGState* st, double* partials, const double* b, const double* q,
                    const double* diag, double* x, double* r, double* d, double* qi,
                    const uint8_t* bmask, int zero_guess, double rel_tol, int32_t max_hist,
                    double* hist, int64_t n, hipStream_t s);
// alpha = rz / (d . q), d . q from the element energies plus d_b^2 over the essential
// rows (has_ess: a constrained operator); breakdown (done = 2) if d . q <= 0 or alpha
// is not finite; x += alpha d; r -= alpha q; q0 (null: none; may be q) = 0
void launch_cg_update(CGState* st, double* partials, double* epart, int nepart, bool has_ess,
                      double* x, double* r, const double* d, const double* q, const double* diag,
                      double* q0, int64_t n, hipStream_t s);
// rz, rr, beta, iter, hist, convergence; dnew = r / diag + beta d (dnew may be d)
void launch_cg_direction(CGState* st, double* partials, const double* r, const double* diag,
                         const double* d, double* dnew, double* q, const uint8_t* bmask,
                         double* hist, int64_t n, hipStream_t s);
// Flexible CG (done = 3: the preconditioner returned r.z <= 0).  max_hist < 0: a restart
// inside a solve, which keeps the iteration count
void launch_fcg_init(CGState* st, double* partials, const double* b, const double* q, double* x,
                     double* r, int zero_guess, double rel_tol, int32_t max_hist, double* hist,
                     int64_t n, hipStream_t s);
void launch_fcg_start(CGState* st, double* partials, const double* r, const double* z, double* p,
                      double* q, const uint8_t* bmask, int64_t n, hipStream_t s);
// x += alpha p; r -= alpha q; zj = r / diag, and zj = r where bmask (may be null) marks
// the essential rows of a constrained operator (unit diagonal there): the Jacobi part
// of the next preconditioned residual
void launch_fcg_update(CGState* st, double* partials, double* epart, int nepart, double* x,
                       double* r, const double* p, const double* q, const double* diag,
                       const uint8_t* bmask, double* zj, int64_t n, hipStream_t s);
// rr, iter, hist, convergence; r.z and r.z_old
void launch_fcg_beta(CGState* st, double* partials, const double* r, const double* z,
                     const double* zold, double* hist, int64_t n, hipStream_t s);
// beta; p = z + beta p
void launch_fcg_direction(CGState* st, double* partials, const double* z, double* p, double* q,
                          const uint8_t* bmask, int64_t n, hipStream_t s);
// res2 = ||b - q||^2 and, if r is not null, r = b - q (always runs, ignores `done`)
void launch_residual(CGState* st, double* partials, const double* b, const double* q, double* r,
                     int64_t n, hipStream_t s);
// Inner PCG of iterative refinement: residual, preconditioned residual, dots and the
// solution x in FP64; direction d and its image q = A_lo d in FP32; dinv = 1/diag in
// FP32 (null: no preconditioner); ess = essential mask of a constrained operator
// (q_b = d_b) or null.  Every kernel that sets the next direction also writes q's
// apply init, so the apply runs without its own init pass.
// r (FP64 residual) *= 1/s; d = z; state restarted with tol2 = tol^2 rr
void launch_ir_start(CGState* st, double* partials, double* r, double s, const float* dinv,
                     float* d, float* q, const uint8_t* ess, double inner_rel_tol, int64_t n,
                     hipStream_t stream);
// alpha; x += (s alpha) d; r -= alpha q; q0 (null: none; not q) = 0
void launch_ir_update(CGState* st, double* partials, double* epart, int nepart, bool has_ess,
                      double* x, double s, double* r, const float* d, const float* q,
                      const float* dinv, float* q0, int64_t n, hipStream_t stream);
// rz, rr, beta, iter, convergence (replaced: beta as launch_ir_replace left it, nothing
// else changes); dnew = z + beta d (dnew may be d); q = apply init of dnew
void launch_ir_direction(CGState* st, double* partials, bool replaced, const double* r,
                         const float* dinv, const float* d, float* dnew, float* q,
                         const uint8_t* ess, int64_t n, hipStream_t stream);
// Reliable update after a residual replacement: r (the FP64 residual) *= 1/s_new,
// beta = -(z.q)/(d.q) so that launch_ir_direction continues with a direction
// conjugate to the kept one (done = 2 on breakdown)
void launch_ir_replace(CGState* st, double* partials, double* r, double s_new, const float* dinv,
                       const float* d, const float* q, double inner_rel_tol, int64_t n,
                       hipStream_t stream);
// dinv = 1/diag rounded to FP32
void launch_ir_dinv(const double* diag, float* dinv, int64_t n, hipStream_t stream);
// dst = convert(src) to f32 or bf16 (round to nearest even)
void launch_convert(const double* src, void* dst, int dtype, int64_t n, hipStream_t s);

}  // namespace pafem
