// The transposed element restriction G^t and the atomic scatter's start, and the linear form
// on rules other than q1d = p + 2 (a general kernel with runtime sizes: one workgroup per
// element, dynamic LDS).  The other setup kernels are in k_assemble.hip.  FP64.
#include "assemble.hpp"
#include "device.hpp"
#include "launch.hpp"

namespace pafem {

namespace {

#define HIP_LAUNCH_CHECK()                                                        \
  do {                                                                            \
    hipError_t err_ = hipGetLastError();                                          \
    if (err_ != hipSuccess)                                                       \
      throw Error(PAFEM_EHIP, std::string("kernel launch: ") + hipGetErrorString(err_)); \
  } while (0)

struct TabView {
  const double *pts, *wts, *B, *G, *Bg, *Gg;
};

TabView tab_view(const DevSpace& sp, int Q) {
  const int D = sp.p + 1, NG = sp.ng;
  const double* t = sp.tables + table_offset_doubles(Q, D, NG);
  TabView v;
  v.pts = t;
  v.wts = t + Q;
  v.B = t + 2 * Q;
  v.G = v.B + Q * D;
  v.Bg = v.G + Q * D;
  v.Gg = v.Bg + Q * NG;
  return v;
}

// Jacobian J_ab = d x_a / d xhat_b of the element map at quadrature point q, from
// the element's geometry nodes X[k][3] and the 1D geometry tables Bg, Gg [Q][NG].
__device__ void element_jacobian(int q, int Q, int NG, const double* X, const double* Bg,
                                 const double* Gg, double J[3][3], double x[3]) {
  const int q1 = q % Q, q2 = (q / Q) % Q, q3 = q / (Q * Q);
  for (int a = 0; a < 3; ++a) {
    x[a] = 0.0;
    for (int b = 0; b < 3; ++b) J[a][b] = 0.0;
  }
  for (int k3 = 0; k3 < NG; ++k3)
    for (int k2 = 0; k2 < NG; ++k2)
      for (int k1 = 0; k1 < NG; ++k1) {
        const double b1 = Bg[q1 * NG + k1], g1 = Gg[q1 * NG + k1];
        const double b2 = Bg[q2 * NG + k2], g2 = Gg[q2 * NG + k2];
        const double b3 = Bg[q3 * NG + k3], g3 = Gg[q3 * NG + k3];
        const double w = b1 * b2 * b3;
        const double d0 = g1 * b2 * b3, d1 = b1 * g2 * b3, d2 = b1 * b2 * g3;
        const double* Xk = X + 3 * (k1 + NG * (k2 + NG * k3));
        for (int a = 0; a < 3; ++a) {
          x[a] += w * Xk[a];
          J[a][0] += Xk[a] * d0;
          J[a][1] += Xk[a] * d1;
          J[a][2] += Xk[a] * d2;
        }
      }
}

// out[i1,i2,i3] = sum_q T[q1,i1] T[q2,i2] T[q3,i3] in[q1,q2,q3] by three one-axis
// contractions through LDS (sum factorization of B^t).
__device__ void contract_to_dofs(int Q, int D, const double* in, double* t1, double* t2,
                                 double* out, const double* T) {
  const int nt = blockDim.x, tid = threadIdx.x;
  for (int idx = tid; idx < Q * Q * D; idx += nt) {
    const int i1 = idx % D, q23 = idx / D;
    double s = 0.0;
    for (int q1 = 0; q1 < Q; ++q1) s += T[q1 * D + i1] * in[q23 * Q + q1];
    t1[idx] = s;
  }
  __syncthreads();
  for (int idx = tid; idx < Q * D * D; idx += nt) {
    const int i1 = idx % D, i2 = (idx / D) % D, q3 = idx / (D * D);
    double s = 0.0;
    for (int q2 = 0; q2 < Q; ++q2) s += T[q2 * D + i2] * t1[(q3 * Q + q2) * D + i1];
    t2[idx] = s;
  }
  __syncthreads();
  for (int idx = tid; idx < D * D * D; idx += nt) {
    const int i1 = idx % D, i2 = (idx / D) % D, i3 = idx / (D * D);
    double s = 0.0;
    for (int q3 = 0; q3 < Q; ++q3) s += T[q3 * D + i3] * t2[(q3 * D + i2) * D + i1];
    out[idx] = s;
  }
  __syncthreads();
}

__global__ void linear_form_kernel(const double* __restrict__ gnodes,
                                   const int32_t* __restrict__ orig, int NG, TabView tv, int Q,
                                   int D, int source, const double* __restrict__ fqp,
                                   double scale, double* __restrict__ ye) {
  extern __shared__ double smem[];
  const int e = blockIdx.x;
  const int NN = NG * NG * NG, QQQ = Q * Q * Q, DDD = D * D * D;
  double* sX = smem;
  double* sBg = sX + 3 * NN;
  double* sGg = sBg + Q * NG;
  double* sB = sGg + Q * NG;
  double* sF = sB + Q * D;
  double* t1 = sF + QQQ;
  double* t2 = t1 + Q * Q * D;
  double* out = t2 + Q * D * D;
  for (int i = threadIdx.x; i < 3 * NN; i += blockDim.x) sX[i] = gnodes[size_t(e) * 3 * NN + i];
  for (int i = threadIdx.x; i < Q * NG; i += blockDim.x) {
    sBg[i] = tv.Bg[i];
    sGg[i] = tv.Gg[i];
  }
  for (int i = threadIdx.x; i < Q * D; i += blockDim.x) sB[i] = tv.B[i];
  __syncthreads();
  const double pi = 3.14159265358979323846;
  for (int q = threadIdx.x; q < QQQ; q += blockDim.x) {
    double J[3][3], x[3];
    element_jacobian(q, Q, NG, sX, sBg, sGg, J, x);
    const double det = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
                       J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
                       J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
    const int q1 = q % Q, q2 = (q / Q) % Q, q3 = q / (Q * Q);
    const double w = tv.wts[q1] * tv.wts[q2] * tv.wts[q3];
    double f;
    if (source == PAFEM_SOURCE_ARRAY)
      f = scale * fqp[size_t(orig[e]) * QQQ + q];
    else if (source == PAFEM_SOURCE_CONST)
      f = scale;
    else
      f = scale * 3.0 * pi * pi * sin(pi * x[0]) * sin(pi * x[1]) * sin(pi * x[2]);
    sF[q] = w * det * f;
  }
  __syncthreads();
  contract_to_dofs(Q, D, sF, t1, t2, out, sB);
  for (int i = threadIdx.x; i < DDD; i += blockDim.x) ye[size_t(e) * DDD + i] = out[i];
}

template <typename T>
__global__ void evec_gather_kernel(const int32_t* __restrict__ toff,
                                   const int32_t* __restrict__ tidx,
                                   const uint8_t* __restrict__ bmask, const T* __restrict__ ye,
                                   const T* __restrict__ x, int bc_mode, T bc_value,
                                   T* __restrict__ y, int64_t n) {
  for (int64_t g = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; g < n;
       g += int64_t(gridDim.x) * blockDim.x) {
    if (bc_mode != 0 && bmask[g]) {
      y[g] = (bc_mode == 1) ? x[g] : bc_value;
      continue;
    }
    // four entries at a time: their loads in flight together, the sum in index order
    T s = T(0);
    const int32_t k1 = toff[g + 1];
    for (int32_t k = toff[g]; k < k1; k += 4) {
      int32_t i[4];
      T v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) i[j] = tidx[min(k + j, k1 - 1)];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = ye[i[j]];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + j < k1) s += v[j];
    }
    y[g] = s;
  }
}

// y = x on the essential dofs (constrained), 0 on the others; blockIdx.y: component, at
// stride n.  One launch for all dofs and components, four dofs per thread, NP of them
// neighbours with one load of their masks and one store (NP > 1: 16 bytes, for which x, y and
// every component have to be aligned; the thread that finds fewer than NP left takes them one
// by one).  All masks are loaded before the first is looked at.  45000 dofs 2.8 -> 2.4 us, 3.9M
// 8.7 -> 7.8, 29M 69 -> 57 (one dof at a time, 8-byte stores -> this).
template <typename T, int NP>
__global__ void __launch_bounds__(256)
    scatter_init_kernel(const uint8_t* __restrict__ bmask, const T* __restrict__ x,
                        int constrained, T* __restrict__ y, int64_t n) {
  typedef T pack __attribute__((ext_vector_type(NP)));
  typedef uint8_t mask __attribute__((ext_vector_type(NP)));
  const int64_t off = int64_t(blockIdx.y) * n;
  const int64_t g0 = int64_t(blockIdx.x) * (4 * 256) + NP * threadIdx.x;
  constexpr int K = 4 / NP;
  mask m[K];
  pack v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t g = g0 + k * (256 * NP);
    m[k] = uint8_t(0);
    if (constrained && g + NP <= n) m[k] = *reinterpret_cast<const mask*>(bmask + g);
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    bool any = false;
#pragma unroll
    for (int j = 0; j < NP; ++j) any = any || m[k][j];
    v[k] = T(0);
    if (any) v[k] = *reinterpret_cast<const pack*>(x + off + g0 + k * (256 * NP));
  }
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const int64_t g = g0 + k * (256 * NP);
#pragma unroll
    for (int j = 0; j < NP; ++j) v[k][j] = m[k][j] ? v[k][j] : T(0);
    if (g + NP <= n)
      *reinterpret_cast<pack*>(y + off + g) = v[k];
    else
      for (int64_t i = g; i < n; ++i) y[off + i] = (constrained && bmask[i]) ? x[off + i] : T(0);
  }
}

// the same on a list of dofs (~g if essential)
template <typename T>
__global__ void __launch_bounds__(256)
    scatter_init_list_kernel(const int32_t* __restrict__ list, int64_t nl,
                             const T* __restrict__ x, int constrained, T* __restrict__ y,
                             int64_t n) {
  const int64_t off = int64_t(blockIdx.y) * n;
  const int64_t k = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (k >= nl) return;
  const int32_t s = list[k];
  const int64_t g = off + (s < 0 ? ~s : s);
  y[g] = (constrained && s < 0) ? x[g] : T(0);
}

int grid_for(int64_t n, int block) {
  int64_t g = (n + block - 1) / block;
  if (g > (1 << 20)) g = 1 << 20;
  return int(g < 1 ? 1 : g);
}

}  // namespace

void launch_qdata(const DevSpace& sp, int kind, int q1d, const double* coeff, double scale,
                  double* qd, hipStream_t st) {
  if (sp.dim == 2) {
    launch_qdata_2d(sp, kind, q1d, coeff, scale, qd, st);
    HIP_LAUNCH_CHECK();
    return;
  }
  launch_qdata_tiles(sp, kind, q1d, coeff, scale, qd, st);
}

void launch_linear_form_evec(const DevSpace& sp, int q1d, int source, const double* fqp,
                             double scale, double* ye, hipStream_t st) {
  if (sp.dim == 2) {
    launch_linear_form_evec_2d(sp, q1d, source, fqp, scale, ye, st);
    HIP_LAUNCH_CHECK();
    return;
  }
  if (q1d == sp.p + 2) {
    launch_linear_form_tiles(sp, source, fqp, scale, ye, st);
    return;
  }
  const TabView tv = tab_view(sp, q1d);
  const int NN = sp.ng * sp.ng * sp.ng, Q = q1d, D = sp.p + 1;
  const size_t lds = sizeof(double) * (3 * NN + 2 * Q * sp.ng + Q * D + Q * Q * Q + Q * Q * D +
                                       Q * D * D + D * D * D);
  hipLaunchKernelGGL(linear_form_kernel, dim3(unsigned(sp.ne)), dim3(256), lds, st, sp.gnodes,
                     sp.elem_orig, sp.ng, tv, Q, D, source, fqp, scale, ye);
  HIP_LAUNCH_CHECK();
}

void launch_diagonal_evec(const DevSpace& sp, int kind, int q1d, const double* qd, double* ye,
                          hipStream_t st) {
  if (sp.dim == 2) {
    launch_diagonal_evec_2d(sp, kind, q1d, qd, ye, st);
    HIP_LAUNCH_CHECK();
    return;
  }
  if (q1d != sp.p + 2)
    throw Error(PAFEM_EUNSUPPORTED, "diagonal: operators have q1d = p + 2");
  launch_diagonal_tiles(sp, kind, qd, ye, st);
}

void launch_evec_gather(const DevSpace& sp, const double* ye, const double* x, int bc_mode,
                        double bc_value, double* y, hipStream_t st) {
  hipLaunchKernelGGL(evec_gather_kernel<double>, dim3(grid_for(sp.ndofs, 256)), dim3(256), 0, st,
                     sp.toff, sp.tidx, sp.bmask, ye, x, bc_mode, bc_value, y, sp.ndofs);
  HIP_LAUNCH_CHECK();
}

void launch_evec_gather_f32(const DevSpace& sp, const float* ye, const float* x, int bc_mode,
                            float* y, hipStream_t st) {
  hipLaunchKernelGGL(evec_gather_kernel<float>, dim3(grid_for(sp.ndofs, 256)), dim3(256), 0, st,
                     sp.toff, sp.tidx, sp.bmask, ye, x, bc_mode, 0.0f, y, sp.ndofs);
  HIP_LAUNCH_CHECK();
}

namespace {
template <typename T>
void scatter_init(const DevSpace& sp, const T* x, bool constrained, T* y, hipStream_t st,
                  int ncomp, bool skip_private) {
  if (skip_private) {
    const int64_t nl = sp.nshared;
    if (nl > 0)
      hipLaunchKernelGGL(scatter_init_list_kernel<T>, dim3(unsigned((nl + 255) / 256), ncomp),
                         dim3(256), 0, st, sp.shared, nl, x, int(constrained), y,
                         int64_t(sp.ndofs));
    HIP_LAUNCH_CHECK();
    return;
  }
  // Without constraints the components are one run of zeros, and neither x nor the masks are
  // read (three components of 118k dofs, an odd stride: 2.9 -> 2.6 us, as a plain fill).
  const int nc = constrained ? ncomp : 1;
  const int64_t n = constrained ? sp.ndofs : ncomp * sp.ndofs;
  const dim3 grid(unsigned((n + 1023) / 1024), nc);
  constexpr int NP = 16 / sizeof(T);
  auto aligned = [](const void* p, uintptr_t a) { return reinterpret_cast<uintptr_t>(p) % a == 0; };
  const bool packs = aligned(y, 16) && (!constrained || (aligned(x, 16) && aligned(sp.bmask, NP) &&
                                                         (nc == 1 || n % NP == 0)));
  if (packs)
    hipLaunchKernelGGL((scatter_init_kernel<T, NP>), grid, dim3(256), 0, st, sp.bmask, x,
                       int(constrained), y, n);
  else
    hipLaunchKernelGGL((scatter_init_kernel<T, 1>), grid, dim3(256), 0, st, sp.bmask, x,
                       int(constrained), y, n);
  HIP_LAUNCH_CHECK();
}
}  // namespace

void launch_scatter_init(const DevSpace& sp, const double* x, bool constrained, double* y,
                         hipStream_t st, int ncomp, bool skip_private) {
  scatter_init(sp, x, constrained, y, st, ncomp, skip_private);
}

void launch_scatter_init(const DevSpace& sp, const float* x, bool constrained, float* y,
                         hipStream_t st) {
  scatter_init(sp, x, constrained, y, st, 1, false);
}

}  // namespace pafem
