// Assembly kernels on the apply's tiles: the quadrature data, the element diagonals and the
// element load vectors of hexahedra ("Operator Decomposition": D, and B^t of the point
// values), as a program runs them again for every new coefficient or source.
//
// One workgroup = one tile of the tile-interleaved quadrature data, Q*Q threads per
// element: a thread owns the z-line (qy, qx), so every load and store of quadrature data
// is one contiguous run of the workgroup (16 bytes per thread where the components are
// paired), the geometry nodes are contracted over (qx, qy) once per thread instead of once
// per point, and the transposed contractions go one 1D line per thread as in the fused
// apply (k_apply.hip), their arrays in one LDS region per element, written in place.
//
// These are bound by the quadrature data and the element vectors in HBM.  At p = 3 on 40^3
// elements (one workgroup per element, one thread per point and stage output before):
// quadrature data 239 -> 151 us, diagonal 517 -> 103, load vector 247 -> 67 (with the
// gathers and the call); at p = 1 on 100^3 the diagonal 5904 -> 259.
#include "assemble.hpp"
#include "device.hpp"

namespace pafem {

namespace {

void check_launch(const char* what) {
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess)
    throw Error(PAFEM_EHIP, std::string(what) + ": " + hipGetErrorString(err));
}

// The element map of one z-line: geometry nodes contracted over (qx, qy), per node layer
// k3 and coordinate a: value, x-derivative, y-derivative.
template <int NG>
struct LineMap {
  double v[3][NG], dx[3][NG], dy[3][NG];

  // X [k3][k2][k1][a], k1 fastest
  __device__ __forceinline__ void load(const double* __restrict__ X, const double* __restrict__ Bg,
                                       const double* __restrict__ Gg, int qx, int qy) {
    double b1[NG], g1[NG];
#pragma unroll
    for (int k = 0; k < NG; ++k) {
      b1[k] = Bg[qx * NG + k];
      g1[k] = Gg[qx * NG + k];
    }
#pragma unroll
    for (int k3 = 0; k3 < NG; ++k3) {
#pragma unroll
      for (int a = 0; a < 3; ++a) v[a][k3] = dx[a][k3] = dy[a][k3] = 0.0;
#pragma unroll
      for (int k2 = 0; k2 < NG; ++k2) {
        const double b2 = Bg[qy * NG + k2], g2 = Gg[qy * NG + k2];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          double s = 0.0, d = 0.0;
#pragma unroll
          for (int k1 = 0; k1 < NG; ++k1) {
            const double xa = X[3 * (k1 + NG * (k2 + NG * k3)) + a];
            s += b1[k1] * xa;
            d += g1[k1] * xa;
          }
          v[a][k3] += b2 * s;
          dx[a][k3] += b2 * d;
          dy[a][k3] += g2 * s;
        }
      }
    }
  }

  // J[a][b] = d x_a / d xhat_b at plane qz, and the point itself
  __device__ __forceinline__ void at(const double* __restrict__ Bg, const double* __restrict__ Gg,
                                     int qz, double J[3][3], double x[3]) const {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double j0 = 0.0, j1 = 0.0, j2 = 0.0, p = 0.0;
#pragma unroll
      for (int k = 0; k < NG; ++k) {
        const double b = Bg[qz * NG + k], g = Gg[qz * NG + k];
        j0 += b * dx[a][k];
        j1 += b * dy[a][k];
        j2 += g * v[a][k];
        p += b * v[a][k];
      }
      J[a][0] = j0;
      J[a][1] = j1;
      J[a][2] = j2;
      x[a] = p;
    }
  }
};

// NC values of one point into the tile layout: qe = the tile's data plus this thread's
// point, plane = values of one component and plane of the tile
template <int NC>
__device__ __forceinline__ void put_point(double* __restrict__ qd, size_t tile, int tid, int Q,
                                          int qz, int plane, const double* v) {
  double* const t = qd + tile * NC * Q * plane;
  if constexpr (NC % 6 == 0) {
#pragma unroll
    for (int k = 0; k < NC / 2; ++k) {
      pafem_d2 w;
      w.x = v[2 * k];
      w.y = v[2 * k + 1];
      *reinterpret_cast<pafem_d2*>(t + size_t(k * Q + qz) * plane * 2 + 2 * tid) = w;
    }
  } else {
#pragma unroll
    for (int c = 0; c < NC; ++c) t[size_t(c * Q + qz) * plane + tid] = v[c];
  }
}

template <int NG>
__global__ void __launch_bounds__(256)
    qdata_tile_kernel(const double* __restrict__ gnodes, const int32_t* __restrict__ orig,
                      const double* __restrict__ wts, const double* __restrict__ Bg,
                      const double* __restrict__ Gg, int Q, int kind,
                      const double* __restrict__ coeff, double scale, double* __restrict__ qd,
                      int32_t* status, int ne) {
  const int QQ = Q * Q, tid = threadIdx.x, plane = blockDim.x;
  const int el = tid / QQ, r = tid - el * QQ;
  const size_t tile = blockIdx.x;
  const int64_t e = int64_t(tile) * (plane / QQ) + el;
  if (e >= ne) return;
  const int qy = r / Q, qx = r - qy * Q;
  const int32_t oe = orig[e];
  const size_t p0 = size_t(oe) * QQ * Q + r;  // this line's first point, caller order
  LineMap<NG> map;
  map.load(gnodes + size_t(e) * (NG * NG * NG * 3), Bg, Gg, qx, qy);
  const double wxy = wts[qx] * wts[qy];
  for (int qz = 0; qz < Q; ++qz) {
    double J[3][3], x[3];
    map.at(Bg, Gg, qz, J, x);
    // adjugate A = det(J) J^{-1}
    double A[3][3];
    A[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
    A[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
    A[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
    A[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
    A[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
    A[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
    A[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
    A[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
    A[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
    const double det = J[0][0] * A[0][0] + J[0][1] * A[1][0] + J[0][2] * A[2][0];
    if (!(det > 0.0)) atomicMin(status, oe);
    const double w = wxy * wts[qz];
    const size_t pt = p0 + size_t(qz) * QQ;
    auto gram = [&](const double M[3][3], bool rows, double f, double* v) {
      // f M M^T (rows) or f M^T M, entries 00 01 02 11 12 22
      int k = 0;
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = a; b < 3; ++b, ++k)
          v[k] = rows ? f * (M[a][0] * M[b][0] + M[a][1] * M[b][1] + M[a][2] * M[b][2])
                      : f * (M[0][a] * M[0][b] + M[1][a] * M[1][b] + M[2][a] * M[2][b]);
    };
    double v[12];
    switch (kind) {
      case PAFEM_MASS:
        v[0] = w * (scale * (coeff ? coeff[pt] : 1.0)) * det;
        put_point<1>(qd, tile, tid, Q, qz, plane, v);
        break;
      case PAFEM_DIFFUSION_GEOM:  // the apply recomputes the geometric part
        v[0] = w * (scale * (coeff ? coeff[pt] : 1.0));
        put_point<1>(qd, tile, tid, Q, qz, plane, v);
        break;
      case PAFEM_GRADIENT:
      case PAFEM_DIVERGENCE: {
        // w kappa det J J^{-T} as D[c][b] = w kappa adj(J)[b][c]: physical derivative c
        // (the gradient's output component, the divergence's input component),
        // reference derivative b
        const double f = w * (scale * (coeff ? coeff[pt] : 1.0));
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
          for (int b = 0; b < 3; ++b) v[3 * c + b] = f * A[b][c];
        put_point<9>(qd, tile, tid, Q, qz, plane, v);
        break;
      }
      case PAFEM_ELASTICITY: {
        // J^{-1} = A / det J as [b][d] = d xhat_b / d x_d, then w det J lambda and
        // w det J mu, lambda and mu from the point's coefficient pair
        const double id = 1.0 / det, wd = scale * w * det;
#pragma unroll
        for (int b = 0; b < 3; ++b)
#pragma unroll
          for (int d = 0; d < 3; ++d) v[3 * b + d] = A[b][d] * id;
        v[9] = wd * coeff[2 * pt];
        v[10] = wd * coeff[2 * pt + 1];
        put_point<11>(qd, tile, tid, Q, qz, plane, v);
        break;
      }
      case PAFEM_CONVECTION:
      case PAFEM_DG_CONVECTION: {
        // alpha det J J^{-1} beta = alpha adj(J) beta, beta = scale * velocity at the point
        // (the DG convection: one constant velocity)
        const double* const vel = kind == PAFEM_DG_CONVECTION ? coeff : coeff + 3 * pt;
        const double b0 = scale * vel[0], b1 = scale * vel[1], b2 = scale * vel[2];
#pragma unroll
        for (int b = 0; b < 3; ++b) v[b] = w * (A[b][0] * b0 + A[b][1] * b1 + A[b][2] * b2);
        put_point<3>(qd, tile, tid, Q, qz, plane, v);
        break;
      }
      case PAFEM_HCURL_MAXWELL:
        // curl-curl w alpha J^T J / det J (the reference curl maps with J / det J), then
        // the mass part w beta A A^T / det J, (alpha, beta) the point's coefficient pair
        gram(J, false, w * (scale * coeff[2 * pt]) / det, v);
        gram(A, true, w * (scale * coeff[2 * pt + 1]) / det, v + 6);
        put_point<12>(qd, tile, tid, Q, qz, plane, v);
        break;
      case PAFEM_HCURL_CURLCURL:
        gram(J, false, w * (scale * (coeff ? coeff[pt] : 1.0)) / det, v);
        put_point<6>(qd, tile, tid, Q, qz, plane, v);
        break;
      default:
        // diffusion and the H(curl) mass: alpha kappa det J J^{-1} J^{-T} = alpha kappa
        // A A^T / det J
        gram(A, true, w * (scale * (coeff ? coeff[pt] : 1.0)) / det, v);
        put_point<6>(qd, tile, tid, Q, qz, plane, v);
    }
  }
}

// diag_i = sum_q sum_ab D_ab(q) d_a phi_i(q) d_b phi_i(q): each (a, b) term is a tensor
// contraction with elementwise products of the 1D tables (B o B, B o G, G o G per axis).
// The six terms go in two passes, by their table along x: 00 (G o G), 01 and 02 (B o G);
// then 11, 12 and 22 (B o B); three arrays in LDS at a time, two or one after the y-lines.
template <int P, bool DIFF>
__global__ void __launch_bounds__(qdata_tile(P + 2) * (P + 2) * (P + 2))
    diagonal_tile_kernel(const double* __restrict__ tabB, const double* __restrict__ tabG,
                         const double* __restrict__ qd, double* __restrict__ ye, int ne) {
  constexpr int Q = P + 2, D = P + 1, QQ = Q * Q, NE = qdata_tile(Q), LC = D | 1;
  constexpr int NA = DIFF ? 3 : 1, NC = DIFF ? 6 : 1;
  __shared__ double sW[NE * NA * QQ * LC];
  const int tid = threadIdx.x, el = tid / QQ, r = tid - el * QQ;
  const size_t tile = blockIdx.x;
  const int64_t e = int64_t(tile) * NE + el;
  const bool act = e < ne;
  double* const W = sW + el * (NA * QQ * LC);
  // entry (c, qy, qx, dz); y-line outputs (a, dz, dy, qx) at c*Q + qy = a*D + dy
  auto at = [&](int c, int qy, int qx, int dz) -> double& {
    return W[((c * Q + qy) * Q + qx) * LC + dz];
  };
  auto rows = [&](int a, int dy, int qx, int dz) -> double& {
    return at((a * D + dy) / Q, (a * D + dy) % Q, qx, dz);
  };
  const int l0 = r % Q, l1 = r / Q;          // z-line (qx, qy), y-line (qx, dz)
  const int xy = r % D, xz = r / D;          // x-line (dy, dz)
  const bool yline = act && r < D * Q, xline = act && r < D * D;

  // D of this thread's line: all of it up front at p <= 4; above, 6 Q values take the
  // registers of a second wave, so each pass loads its two pairs plane by plane (the
  // middle pair twice)
  constexpr bool STREAM = DIFF && P >= 5;
  const double* const qe = qd + tile * (size_t(NC) * Q * NE * QQ);
  double dq[Q][NC];
  auto load = [&](int qz, int k0, int k1) {
    if constexpr (DIFF) {
#pragma unroll
      for (int k = k0; k < k1; ++k)
        load_pair<double, double>(qe + 2 * (size_t(k * Q + qz) * (NE * QQ) + tid), dq[qz][2 * k],
                                  dq[qz][2 * k + 1]);
    } else {
      dq[qz][0] = load_value<double, double>(qe + qz * (NE * QQ) + tid);
    }
  };
  if (act && !STREAM) {
#pragma unroll
    for (int qz = 0; qz < Q; ++qz) load(qz, 0, 3);
  }
  // at p >= 5 the table entries of a loop iteration are loaded in it: all of them up front
  // outgrow the scalar registers
  auto tab = [&](const double* t) {
    if constexpr (P >= 5)
      return opaque_ptr(t);
    else
      return t;
  };
  double acc[D];
#pragma unroll
  for (int dx = 0; dx < D; ++dx) acc[dx] = 0.0;

  auto pass = [&](auto second) {
    constexpr bool SECOND = decltype(second)::value;
    constexpr int NY = DIFF && !SECOND ? 2 : 1;  // arrays after the y-lines
    if (act) {
      double t[NA][D];
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int dz = 0; dz < D; ++dz) t[a][dz] = 0.0;
      if (STREAM) load(0, SECOND ? 1 : 0, SECOND ? 3 : 2);
#pragma unroll
      for (int qz = 0; qz < Q; ++qz) {
        const auto rb = tab(tabB + qz * D), rg = tab(tabG + qz * D);
        if constexpr (STREAM) {
          if (qz + 1 < Q) load(qz + 1, SECOND ? 1 : 0, SECOND ? 3 : 2);
          __asm__ volatile("" ::: "memory");  // keep the next plane's loads in this iteration
        }
#pragma unroll
        for (int dz = 0; dz < D; ++dz) {
          const double b = rb[dz], g = rg[dz];
          if constexpr (!DIFF) {
            t[0][dz] += b * b * dq[qz][0];
          } else if constexpr (!SECOND) {
            t[0][dz] += b * b * dq[qz][0];
            t[1][dz] += b * b * dq[qz][1];
            t[2][dz] += b * g * dq[qz][2];
          } else {
            t[0][dz] += b * b * dq[qz][3];
            t[1][dz] += b * g * dq[qz][4];
            t[2][dz] += g * g * dq[qz][5];
          }
        }
      }
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int dz = 0; dz < D; ++dz) at(a, l1, l0, dz) = t[a][dz];
    }
    __syncthreads();
    if (yline) {
      double in[NA][Q];
#pragma unroll
      for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int qy = 0; qy < Q; ++qy) in[a][qy] = at(a, qy, l0, l1);
#pragma unroll
      for (int dy = 0; dy < D; ++dy) {
        const auto cb = tab(tabB + dy), cg = tab(tabG + dy);
        double o[NY];
#pragma unroll
        for (int a = 0; a < NY; ++a) o[a] = 0.0;
#pragma unroll
        for (int qy = 0; qy < Q; ++qy) {
          const double b = cb[qy * D], g = cg[qy * D];
          if constexpr (!DIFF) {
            o[0] += b * b * in[0][qy];
          } else if constexpr (!SECOND) {
            o[0] += b * b * in[0][qy];
            o[1] += 2.0 * (b * g * in[1][qy] + b * b * in[2][qy]);
          } else {
            o[0] += g * g * in[0][qy] + 2.0 * (b * g * in[1][qy]) + b * b * in[2][qy];
          }
        }
#pragma unroll
        for (int a = 0; a < NY; ++a) rows(a, dy, l0, l1) = o[a];
      }
    }
    __syncthreads();
    if (xline) {
#pragma unroll
      for (int qx = 0; qx < Q; ++qx) {
        const auto rb = tab(tabB + qx * D), rg = tab(tabG + qx * D);
        double in[NY];
#pragma unroll
        for (int a = 0; a < NY; ++a) in[a] = rows(a, xy, qx, xz);
#pragma unroll
        for (int dx = 0; dx < D; ++dx) {
          const double b = rb[dx], g = rg[dx];
          if constexpr (NY == 2)
            acc[dx] += g * g * in[0] + b * g * in[1];
          else
            acc[dx] += b * b * in[0];
        }
      }
    }
  };
  pass(std::false_type{});
  if constexpr (DIFF) {
    __syncthreads();  // the x-lines have read the region
    pass(std::true_type{});
  }
  if (xline) {
    double* const out = ye + size_t(e) * (D * D * D) + r * D;
#pragma unroll
    for (int dx = 0; dx < D; ++dx) out[dx] = acc[dx];
  }
}

// B^t (w det J f): the point values of a z-line in registers, then z-, y- and x-lines
// (SINE: the built-in sine source, its planes one after the other: unrolled, the
// argument reductions of 3 Q sines took 154 registers and more)
template <int P, int NG, bool SINE>
__global__ void __launch_bounds__(qdata_tile(P + 2) * (P + 2) * (P + 2))
    linear_form_tile_kernel(const double* __restrict__ gnodes, const int32_t* __restrict__ orig,
                            const double* __restrict__ wts, const double* __restrict__ tabB,
                            const double* __restrict__ Bg, const double* __restrict__ Gg,
                            const double* __restrict__ fqp, double scale,
                            double* __restrict__ ye, int ne) {
  constexpr int Q = P + 2, D = P + 1, QQ = Q * Q, NE = qdata_tile(Q), LC = D | 1;
  __shared__ double sW[NE * QQ * LC];
  const int tid = threadIdx.x, el = tid / QQ, r = tid - el * QQ;
  const int64_t e = int64_t(blockIdx.x) * NE + el;
  const bool act = e < ne;
  double* const W = sW + el * (QQ * LC);
  auto at = [&](int qy, int qx, int dz) -> double& { return W[(qy * Q + qx) * LC + dz]; };
  const int l0 = r % Q, l1 = r / Q;
  const int xy = r % D, xz = r / D;

  if (act) {
    double f[SINE ? 1 : Q];
    if constexpr (!SINE) {
      const double* const fe = fqp ? fqp + size_t(orig[e]) * (QQ * Q) + r : nullptr;
#pragma unroll
      for (int qz = 0; qz < Q; ++qz) f[qz] = fe ? scale * fe[qz * QQ] : scale;
    }
    LineMap<NG> map;
    map.load(gnodes + size_t(e) * (NG * NG * NG * 3), Bg, Gg, l0, l1);
    const double wxy = wts[l0] * wts[l1];
    double t[D];
#pragma unroll
    for (int dz = 0; dz < D; ++dz) t[dz] = 0.0;
    auto point = [&](int qz, double fq) {
      double J[3][3], x[3];
      map.at(Bg, Gg, qz, J, x);
      const double det = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1]) -
                         J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0]) +
                         J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
      if constexpr (SINE) {
        const double pi = 3.14159265358979323846;
        fq = scale * 3.0 * pi * pi * sin(pi * x[0]) * sin(pi * x[1]) * sin(pi * x[2]);
      }
      const double v = wxy * wts[qz] * det * fq;
#pragma unroll
      for (int dz = 0; dz < D; ++dz) t[dz] += tabB[qz * D + dz] * v;
    };
    if constexpr (SINE) {
#pragma unroll 1
      for (int qz = 0; qz < Q; ++qz) point(qz, 0.0);
    } else {
#pragma unroll
      for (int qz = 0; qz < Q; ++qz) point(qz, f[qz]);
    }
#pragma unroll
    for (int dz = 0; dz < D; ++dz) at(l1, l0, dz) = t[dz];
  }
  __syncthreads();
  if (act && r < D * Q) {
    double in[Q];
#pragma unroll
    for (int qy = 0; qy < Q; ++qy) in[qy] = at(qy, l0, l1);
#pragma unroll
    for (int dy = 0; dy < D; ++dy) {
      double o = 0.0;
#pragma unroll
      for (int qy = 0; qy < Q; ++qy) o += tabB[qy * D + dy] * in[qy];
      at(dy, l0, l1) = o;
    }
  }
  __syncthreads();
  if (act && r < D * D) {
    double acc[D];
#pragma unroll
    for (int dx = 0; dx < D; ++dx) acc[dx] = 0.0;
#pragma unroll
    for (int qx = 0; qx < Q; ++qx) {
      const double in = at(xy, qx, xz);
#pragma unroll
      for (int dx = 0; dx < D; ++dx) acc[dx] += tabB[qx * D + dx] * in;
    }
    double* const out = ye + size_t(e) * (D * D * D) + r * D;
#pragma unroll
    for (int dx = 0; dx < D; ++dx) out[dx] = acc[dx];
  }
}

template <int P>
void diagonal_order(const DevSpace& sp, bool diff, const double* qd, double* ye, hipStream_t st) {
  constexpr int Q = P + 2, NE = qdata_tile(Q);
  const unsigned nblk = unsigned((sp.ne + NE - 1) / NE);
  const double* B = sp.tables + table_offset_doubles(Q, P + 1, sp.ng) + 2 * Q;
  const double* G = B + Q * (P + 1);
  if (diff)
    hipLaunchKernelGGL((diagonal_tile_kernel<P, true>), dim3(nblk), dim3(NE * Q * Q), 0, st, B, G,
                       qd, ye, int(sp.ne));
  else
    hipLaunchKernelGGL((diagonal_tile_kernel<P, false>), dim3(nblk), dim3(NE * Q * Q), 0, st, B, G,
                       qd, ye, int(sp.ne));
}

template <int P>
void linear_form_order(const DevSpace& sp, int source, const double* fqp, double scale,
                       double* ye, hipStream_t st) {
  constexpr int Q = P + 2, NE = qdata_tile(Q);
  const unsigned nblk = unsigned((sp.ne + NE - 1) / NE);
  const double* t = sp.tables + table_offset_doubles(Q, P + 1, sp.ng);
  const double *wts = t + Q, *B = t + 2 * Q, *Bg = B + 2 * Q * (P + 1), *Gg = Bg + Q * sp.ng;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(nblk), dim3(NE * Q * Q), 0, st, sp.gnodes, sp.elem_orig, wts,
                       B, Bg, Gg, source == PAFEM_SOURCE_ARRAY ? fqp : nullptr, scale, ye,
                       int(sp.ne));
  };
  const bool sine = source == PAFEM_SOURCE_SINE;
  if (sp.ng == 2)
    sine ? launch(linear_form_tile_kernel<P, 2, true>) : launch(linear_form_tile_kernel<P, 2, false>);
  else
    sine ? launch(linear_form_tile_kernel<P, 3, true>) : launch(linear_form_tile_kernel<P, 3, false>);
}

}  // namespace

void launch_qdata_tiles(const DevSpace& sp, int kind, int q1d, const double* coeff, double scale,
                        double* qd, hipStream_t st) {
  const int Q = q1d, D = sp.p + 1, NE = qdata_tile(Q);
  const unsigned nblk = unsigned((sp.ne + NE - 1) / NE);
  const double* t = sp.tables + table_offset_doubles(Q, D, sp.ng);
  const double *wts = t + Q, *Bg = t + 2 * Q + 2 * Q * D, *Gg = Bg + Q * sp.ng;
  if (sp.ng == 2)
    hipLaunchKernelGGL(qdata_tile_kernel<2>, dim3(nblk), dim3(NE * Q * Q), 0, st, sp.gnodes,
                       sp.elem_orig, wts, Bg, Gg, Q, kind, coeff, scale, qd, sp.status,
                       int(sp.ne));
  else
    hipLaunchKernelGGL(qdata_tile_kernel<3>, dim3(nblk), dim3(NE * Q * Q), 0, st, sp.gnodes,
                       sp.elem_orig, wts, Bg, Gg, Q, kind, coeff, scale, qd, sp.status,
                       int(sp.ne));
  check_launch("quadrature data");
}

#define PAFEM_ORDERS(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

void launch_diagonal_tiles(const DevSpace& sp, int kind, const double* qd, double* ye,
                           hipStream_t st) {
  switch (sp.p) {
#define PAFEM_CASE(P) \
  case P: diagonal_order<P>(sp, kind != PAFEM_MASS, qd, ye, st); break;
    PAFEM_ORDERS(PAFEM_CASE)
#undef PAFEM_CASE
    default: throw Error(PAFEM_EUNSUPPORTED, "diagonal: order not built");
  }
  check_launch("diagonal");
}

void launch_linear_form_tiles(const DevSpace& sp, int source, const double* fqp, double scale,
                              double* ye, hipStream_t st) {
  switch (sp.p) {
#define PAFEM_CASE(P) \
  case P: linear_form_order<P>(sp, source, fqp, scale, ye, st); break;
    PAFEM_ORDERS(PAFEM_CASE)
#undef PAFEM_CASE
    default: throw Error(PAFEM_EUNSUPPORTED, "linear form: order not built");
  }
  check_launch("linear form");
}

}  // namespace pafem
