// Upwind DG convection on a discontinuous nodal space of hexahedra (convection "including
// DG" among the partially assembled integrators of "GPU Acceleration"): the volume and the
// face terms in one kernel, and the setup of the face values.
//
// With the Gauss-Lobatto nodes the trace of an element function on one of its faces
// depends only on the (p+1)^2 dofs of that face, so an element needs no more of a
// neighbour than those.  At each Gauss point of a face the upwind value times the stored
// w (beta . N) is formed (the neighbour's points reached through the face's orientation)
// and contracted back onto the element's face dofs.  Boundary faces keep the outflow part
// only (zero inflow data).
#include "device.hpp"
#include "launch.hpp"

namespace pafem {

namespace {

#define HIP_LAUNCH_CHECK_DG()                                                     \
  do {                                                                            \
    hipError_t err_ = hipGetLastError();                                          \
    if (err_ != hipSuccess)                                                       \
      throw Error(PAFEM_EHIP, std::string("kernel launch: ") + hipGetErrorString(err_)); \
  } while (0)

// tangential axes of face f = 2 a + side, in increasing order
__host__ __device__ inline void face_axes(int f, int& a, int& b, int& c) {
  a = f / 2;
  b = (a == 0) ? 1 : 0;
  c = (a == 2) ? 1 : 2;
}

// index of the "+" side's point / node for the "-" side's (is, it) on an n x n grid
__device__ inline int face_perm(int orient, int is, int it, int n) {
  int u, v;
  if (orient & 1) {
    u = it;
    v = is;
  } else {
    u = is;
    v = it;
  }
  if (orient & 2) u = n - 1 - u;
  if (orient & 4) v = n - 1 - v;
  return u + n * v;
}

// 1D Lagrange basis on NG equispaced nodes of [0, 1]: value and derivative of node j at x
__device__ inline void geom_basis(int NG, int j, double x, double& val, double& der) {
  const double xj = double(j) / (NG - 1);
  val = 1.0;
  der = 0.0;
  for (int m = 0; m < NG; ++m) {
    if (m == j) continue;
    const double xm = double(m) / (NG - 1);
    double prod = 1.0 / (xj - xm);
    for (int l = 0; l < NG; ++l)
      if (l != j && l != m) prod *= (x - double(l) / (NG - 1)) / (xj - double(l) / (NG - 1));
    der += prod;
    val *= (x - xm) / (xj - xm);
  }
}

// w_s w_t scale (beta . N) at the Q x Q Gauss points of every face, N = T_b x T_c
// oriented outward from the face's first element (the interior face's "-" side); after
// them, one 8-byte slot per face with its two elements' caller indices, part of the data's
// published layout (pafem.h; the apply takes its neighbours from the space)
__global__ void dg_face_qdata_kernel(const int32_t* __restrict__ faces,
                                     const int32_t* __restrict__ bfaces, int64_t nf, int64_t nb,
                                     const int32_t* __restrict__ orig,
                                     const double* __restrict__ gnodes, int NG,
                                     const double* __restrict__ pts,
                                     const double* __restrict__ wts, int Q,
                                     const double* __restrict__ beta3, double scale,
                                     double* __restrict__ fq) {
  const int64_t g = blockIdx.x;
  if (g >= nf + nb) return;
  int e, f;
  if (g < nf) {
    e = faces[g * kFaceInts + 0];
    f = faces[g * kFaceInts + 2] & 7;
  } else {
    e = bfaces[(g - nf) * 2 + 0];
    f = bfaces[(g - nf) * 2 + 1];
  }
  if (threadIdx.x == 0) {
    int2 o;
    o.x = orig[e];
    o.y = g < nf ? orig[faces[g * kFaceInts + 1]] : 0;
    reinterpret_cast<int2*>(fq + (nf + nb) * Q * Q)[g] = o;
  }
  int a, b, c;
  face_axes(f, a, b, c);
  const int side = f & 1;
  const double* X = gnodes + size_t(e) * NG * NG * NG * 3;
  const double be0 = scale * beta3[0], be1 = scale * beta3[1], be2 = scale * beta3[2];
  // (a, b, c) cyclic: T_b x T_c points along +e_a for the reference cube
  const double sgn = ((a == 1) ? -1.0 : 1.0) * (side ? 1.0 : -1.0);
  for (int q = threadIdx.x; q < Q * Q; q += blockDim.x) {
    const int qs = q % Q, qt = q / Q;
    double xi[3];
    xi[a] = side;
    xi[b] = pts[qs];
    xi[c] = pts[qt];
    double Tb[3] = {0, 0, 0}, Tc[3] = {0, 0, 0};
    for (int k3 = 0; k3 < NG; ++k3)
      for (int k2 = 0; k2 < NG; ++k2)
        for (int k1 = 0; k1 < NG; ++k1) {
          const int kk[3] = {k1, k2, k3};
          double v[3], d[3];
          for (int t = 0; t < 3; ++t) geom_basis(NG, kk[t], xi[t], v[t], d[t]);
          double wb = d[b], wc = d[c];
          for (int t = 0; t < 3; ++t) {
            if (t != b) wb *= v[t];
            if (t != c) wc *= v[t];
          }
          const double* Xk = X + 3 * (k1 + NG * (k2 + NG * k3));
          for (int t = 0; t < 3; ++t) {
            Tb[t] += wb * Xk[t];
            Tc[t] += wc * Xk[t];
          }
        }
    const double N0 = Tb[1] * Tc[2] - Tb[2] * Tc[1];
    const double N1 = Tb[2] * Tc[0] - Tb[0] * Tc[2];
    const double N2 = Tb[0] * Tc[1] - Tb[1] * Tc[0];
    fq[size_t(g) * Q * Q + q] = wts[qs] * wts[qt] * sgn * (be0 * N0 + be1 * N1 + be2 * N2);
  }
}

// One workgroup = one tile of the volume data (k_apply.hip's tiles), Q*Q threads per
// element, everything one 1D line per thread.  Face stages, on the 6 faces of every
// element at once and in the element's own frame of each face:
//   lines (f, j): the D face dofs of both sides, own from LDS, the neighbour's straight from
//                 x into registers through the orientation; contracted to Q values each
//   lines (f, q): the other axis for both sides, the upwind flux at the line's Q points,
//                 contracted back along the same axis in registers
//   lines (f, j): contracted back to the D face dofs, kept in registers
// then the volume term (mass contractions forward, -u (w adj(J) beta) at the points,
// gradient contractions back), the face lines' results added per dof in LDS on the way.
//
// Every interior face is evaluated from both sides (a quarter more arithmetic) so that each
// element writes its own dofs once, with plain stores.  A kernel over the faces, after the
// volume one, added 2 (p+1)^2 FP64 atomics per face, which go to memory one by one: 166 of
// the 266 us at p = 4 on 40^3 elements; fused 131 us.
template <int P>
__global__ void __launch_bounds__(qdata_tile(P + 2) * (P + 2) * (P + 2))
    dg_apply_kernel(const int32_t* __restrict__ gmap, const int4* __restrict__ efaces,
                    const double* __restrict__ tabB, const double* __restrict__ tabG,
                    const double* __restrict__ qd, const double* __restrict__ fq,
                    const double* __restrict__ x, double* __restrict__ y, int ne) {
  constexpr int Q = P + 2, D = P + 1, QQ = Q * Q, DD = D * D, DDD = DD * D;
  constexpr int NE = qdata_tile(Q), NT = NE * QQ;
  constexpr int LC = D | 1, QL = Q | 1;
  constexpr int VOL = 3 * QQ * LC, FACE = 12 * D * QL;
  constexpr int ELEM = VOL > FACE ? VOL : FACE;
  constexpr int RD = (6 * D + QQ - 1) / QQ, RQ = (6 * Q + QQ - 1) / QQ;  // lines per thread
  __shared__ double sW[NE * ELEM];
  __shared__ double sX[NE * DDD];

  const int tid = threadIdx.x, el = tid / QQ, r = tid - el * QQ;
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int e = tile * NE + el;
  const bool act = e < ne;
  double* const W = sW + el * ELEM;
  double* const X = sX + el * DDD;
  auto at = [&](int c, int qy, int qx, int dz) -> double& {
    return W[((c * Q + qy) * Q + qx) * LC + dz];
  };
  // face arrays: side h (0 own, 1 neighbour), line (f, j), q
  auto fa = [&](int h, int f, int j, int q) -> double& { return W[((h * 6 + f) * D + j) * QL + q]; };
  // at p = 8 the table entries are loaded per loop iteration (k_apply.hip)
  auto tab = [&](const double* t) {
    if constexpr (P >= 8)
      return opaque_ptr(t);
    else
      return t;
  };
  auto rowB = [&](int q) { return tab(tabB + q * D); };
  auto rowG = [&](int q) { return tab(tabG + q * D); };
  auto colB = [&](int d) { return tab(tabB + d); };
  auto colG = [&](int d) { return tab(tabG + d); };
  // first dof and strides of the face lines of face f: node (i, j) at base + i si + j sj
  auto face_base = [](int f) { return (f & 1) ? P * (f < 2 ? 1 : f < 4 ? D : DD) : 0; };
  auto stride_i = [](int f) { return f < 2 ? D : 1; };
  auto stride_j = [](int f) { return f < 4 ? DD : D; };

  // Loads return in order: the element's block and its face records before the volume data,
  // behind which x waited for all of it (p = 1, 1e6 elements 276 -> 256 us, p = 4, 64000:
  // 138 -> 131); from p = 6 the volume data last, under the face stages (64.8 -> 61.2 at
  // p = 6 on 20^3, 63.7 -> 62.3 at p = 7 on 17^3; p = 4 on 30^3 slower that way, 64.9 -> 68.9).
  const int own = act ? gmap[size_t(e) * DDD] : 0;
  int4 recs[RD];
#pragma unroll
  for (int k = 0; k < RD; ++k) {
    const int l = r + k * QQ;
    if (act && l < 6 * D) recs[k] = efaces[size_t(e) * 6 + l / D];
  }
  // the volume data of this thread's z-line
  double dq[Q][3];
  auto load_dq = [&]() {
    if (!act) return;
    const double* const qe = qd + size_t(tile) * (3 * Q * NT) + tid;
#pragma unroll
    for (int qz = 0; qz < Q; ++qz)
#pragma unroll
      for (int c = 0; c < 3; ++c) dq[qz][c] = load_value<double, double>(qe + (c * Q + qz) * NT);
  };
  if (P < 6) load_dq();
  // the element's dofs (one contiguous block) into LDS
  if (act)
    for (int i = r; i < DDD; i += QQ) X[i] = x[own + i];
  // the neighbours' face dofs of this thread's lines (f, j), in this element's frame
  double nb[RD][D];
#pragma unroll
  for (int k = 0; k < RD; ++k) {
    const int l = r + k * QQ, f = l / D, j = l - f * D;
#pragma unroll
    for (int i = 0; i < D; ++i) nb[k][i] = 0.0;
    if (act && l < 6 * D) {
      const int4 rec = recs[k];
      if (rec.y >= 0) {
        const int g = (rec.z >> 1) & 7, o = rec.z >> 4;
        // (i, j) -> (u, v): u = i or j, reversed or not; so a line along i is a line there
        const int si = stride_i(g), sj = stride_j(g);
        const int su = (o & 2) ? -si : si, sv = (o & 4) ? -sj : sj;
        const int b0 = rec.y + face_base(g) + ((o & 2) ? P * si : 0) + ((o & 4) ? P * sj : 0);
        const int step = (o & 1) ? sv : su;
        const double* const xn = x + (b0 + j * ((o & 1) ? su : sv));
#pragma unroll
        for (int i = 0; i < D; ++i) nb[k][i] = xn[i * step];
      }
    }
  }
  if (P >= 6) load_dq();
  __syncthreads();

  // face lines (f, j)
#pragma unroll
  for (int k = 0; k < RD; ++k) {
    const int l = r + k * QQ, f = l / D, j = l - f * D;
    if (act && l < 6 * D) {
      double u[D];
      const int b0 = face_base(f) + j * stride_j(f), si = stride_i(f);
#pragma unroll
      for (int i = 0; i < D; ++i) u[i] = X[b0 + i * si];
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const auto rb = rowB(q);
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int i = 0; i < D; ++i) {
          a += rb[i] * u[i];
          b += rb[i] * nb[k][i];
        }
        fa(0, f, j, q) = a;
        fa(1, f, j, q) = b;
      }
    }
  }
  // weights of the lines (f, q), outward from this element; the face's own frame is its
  // "-" element's
  double w[RQ][Q];
  // The sign bit tells the side: 0 takes the own value, 1 the neighbour's.  Where the velocity
  // is tangential both sides take the "+" element's value, so an infinity or NaN of the "-"
  // element does not cross: a zero weight is +0 in the "+" element and -0 in the "-" one.  (A
  // bound per line to compare with costs the registers of a wave at p <= 2: p = 2, 72^3
  // elements, 217 -> 235 us.)
#pragma unroll
  for (int k = 0; k < RQ; ++k) {
    const int l = r + k * QQ, f = l / Q, q = l - f * Q;
    if (act && l < 6 * Q) {
      const int4 rec = efaces[size_t(e) * 6 + f];
      const double* const wf = fq + size_t(rec.x) * QQ;
      const bool plus = rec.z & 1;
#pragma unroll
      for (int t = 0; t < Q; ++t) {
        const double v = 0.0 - wf[plus ? face_perm(rec.z >> 4, q, t, Q) : q + Q * t];  // no -0
        w[k][t] = plus ? v : -v;
      }
    }
  }
  __syncthreads();
  // face lines (f, q): values, upwind flux, back along the same axis
#pragma unroll
  for (int k = 0; k < RQ; ++k) {
    const int l = r + k * QQ, f = l / Q, q = l - f * Q;
    if (act && l < 6 * Q) {
      double a[D], b[D], o[D];
#pragma unroll
      for (int j = 0; j < D; ++j) {
        a[j] = fa(0, f, j, q);
        b[j] = fa(1, f, j, q);
        o[j] = 0.0;
      }
#pragma unroll
      for (int t = 0; t < Q; ++t) {
        const auto rb = rowB(t);
        double va = 0.0, vb = 0.0;
#pragma unroll
        for (int j = 0; j < D; ++j) {
          va += rb[j] * a[j];
          vb += rb[j] * b[j];
        }
        const double F = w[k][t] * (__builtin_signbit(w[k][t]) ? vb : va);
#pragma unroll
        for (int j = 0; j < D; ++j) o[j] += rb[j] * F;
      }
#pragma unroll
      for (int j = 0; j < D; ++j) fa(0, f, j, q) = o[j];
    }
  }
  __syncthreads();
  // face lines (f, j): back to the face dofs, kept in registers until the volume's x-lines
  // have read the element's dofs
  double fv[RD][D];
#pragma unroll
  for (int k = 0; k < RD; ++k) {
    const int l = r + k * QQ, f = l / D, j = l - f * D;
    if (act && l < 6 * D) {
      double in[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) in[q] = fa(0, f, j, q);
#pragma unroll
      for (int i = 0; i < D; ++i) {
        const auto cb = colB(i);
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q) s += cb[q * D] * in[q];
        fv[k][i] = s;
      }
    }
  }
  // volume, along x: thread (dz, dy)
  const bool xline = act && r < DD, yline = act && r < D * Q;
  const int xz = r / D, xy = r - xz * D, l1 = r / Q, l0 = r - l1 * Q;
  double u[D];
  if (xline) {
#pragma unroll
    for (int dx = 0; dx < D; ++dx) u[dx] = X[r * D + dx];
  }
  __syncthreads();  // the face lines have read the region, the x-lines the dofs
  if (xline) {
#pragma unroll
    for (int qx = 0; qx < Q; ++qx) {
      const auto rb = rowB(qx);
      double b = 0.0;
#pragma unroll
      for (int dx = 0; dx < D; ++dx) b += rb[dx] * u[dx];
      at(xy / Q, xy % Q, qx, xz) = b;
    }
  }
  if (act)
    for (int i = r; i < DDD; i += QQ) X[i] = 0.0;
  __syncthreads();
  // the face terms, per dof
#pragma unroll
  for (int k = 0; k < RD; ++k) {
    const int l = r + k * QQ, f = l / D, j = l - f * D;
    if (act && l < 6 * D) {
      const int b0 = face_base(f) + j * stride_j(f), si = stride_i(f);
#pragma unroll
      for (int i = 0; i < D; ++i) atomicAdd(&X[b0 + i * si], fv[k][i]);
    }
  }
  // along y: thread (dz, qx)
  if (yline) {
    double a[D];
#pragma unroll
    for (int dy = 0; dy < D; ++dy) a[dy] = at(dy / Q, dy % Q, l0, l1);
#pragma unroll
    for (int qy = 0; qy < Q; ++qy) {
      const auto rb = rowB(qy);
      double b = 0.0;
#pragma unroll
      for (int dy = 0; dy < D; ++dy) b += rb[dy] * a[dy];
      at(0, qy, l0, l1) = b;
    }
  }
  __syncthreads();
  // along z, the points, back along z: thread (qy, qx)
  if (act) {
    double c[D], t0[D], t1[D], t2[D];
#pragma unroll
    for (int dz = 0; dz < D; ++dz) {
      c[dz] = at(0, l1, l0, dz);
      t0[dz] = t1[dz] = t2[dz] = 0.0;
    }
#pragma unroll
    for (int qz = 0; qz < Q; ++qz) {
      const auto rb = rowB(qz);
      const auto rg = rowG(qz);
      double v = 0.0;
#pragma unroll
      for (int dz = 0; dz < D; ++dz) v += rb[dz] * c[dz];
      const double vx = -dq[qz][0] * v, vy = -dq[qz][1] * v, vz = -dq[qz][2] * v;
#pragma unroll
      for (int dz = 0; dz < D; ++dz) {
        t0[dz] += rb[dz] * vx;
        t1[dz] += rb[dz] * vy;
        t2[dz] += rg[dz] * vz;
      }
    }
#pragma unroll
    for (int dz = 0; dz < D; ++dz) {
      at(0, l1, l0, dz) = t0[dz];
      at(1, l1, l0, dz) = t1[dz];
      at(2, l1, l0, dz) = t2[dz];
    }
  }
  __syncthreads();
  // back along y
  if (yline) {
    double v0[Q], v1[Q], v2[Q];
#pragma unroll
    for (int qy = 0; qy < Q; ++qy) {
      v0[qy] = at(0, qy, l0, l1);
      v1[qy] = at(1, qy, l0, l1);
      v2[qy] = at(2, qy, l0, l1);
    }
#pragma unroll
    for (int dy = 0; dy < D; ++dy) {
      const auto cb = colB(dy);
      const auto cg = colG(dy);
      double b = 0.0, g = 0.0;
#pragma unroll
      for (int qy = 0; qy < Q; ++qy) {
        g += cb[qy * D] * v0[qy];
        b += cg[qy * D] * v1[qy] + cb[qy * D] * v2[qy];
      }
      at(dy / Q, dy % Q, l0, l1) = b;
      at((D + dy) / Q, (D + dy) % Q, l0, l1) = g;
    }
  }
  __syncthreads();
  // back along x, onto the face terms
  if (xline) {
    double wB[Q], wG[Q];
#pragma unroll
    for (int qx = 0; qx < Q; ++qx) {
      wB[qx] = at(xy / Q, xy % Q, qx, xz);
      wG[qx] = at((D + xy) / Q, (D + xy) % Q, qx, xz);
    }
#pragma unroll
    for (int dx = 0; dx < D; ++dx) {
      const auto cb = colB(dx);
      const auto cg = colG(dx);
      double s = 0.0;
#pragma unroll
      for (int qx = 0; qx < Q; ++qx) s += cb[qx * D] * wB[qx] + cg[qx * D] * wG[qx];
      X[r * D + dx] += s;
    }
  }
  __syncthreads();
  if (act)
    for (int i = r; i < DDD; i += QQ) y[own + i] = X[i];
}

template <int P>
void launch_apply_p(const DevSpace& sp, const double* tabB, const double* qd, const double* fq,
                    const double* x, double* y, hipStream_t st) {
  constexpr int Q = P + 2, NE = qdata_tile(Q);
  const unsigned nblk = unsigned((sp.ne + NE - 1) / NE);
  hipLaunchKernelGGL((dg_apply_kernel<P>), dim3(nblk), dim3(NE * Q * Q), 0, st, sp.gmap,
                     reinterpret_cast<const int4*>(sp.efaces), tabB, tabB + Q * (P + 1), qd, fq, x,
                     y, int(sp.ne));
}

}  // namespace

void launch_dg_face_qdata(const DevSpace& sp, int q1d, const double* beta3, double scale,
                          double* fq, hipStream_t st) {
  const int64_t total = sp.nfaces + sp.nbfaces;
  if (total == 0) return;
  const double* t = sp.tables + table_offset_doubles(q1d, sp.p + 1, sp.ng);
  hipLaunchKernelGGL(dg_face_qdata_kernel, dim3(unsigned(total)), dim3(128), 0, st, sp.faces,
                     sp.bfaces, sp.nfaces, sp.nbfaces, sp.elem_orig, sp.gnodes, sp.ng, t, t + q1d,
                     q1d, beta3, scale, fq);
  HIP_LAUNCH_CHECK_DG();
}

void launch_dg_apply(const DevSpace& sp, int q1d, const double* qd, const double* fq,
                     const double* x, double* y, hipStream_t st) {
  if (q1d != sp.p + 2) throw Error(PAFEM_EUNSUPPORTED, "the DG apply is built for q1d = p + 2");
  const double* tabB = sp.tables + table_offset_doubles(q1d, sp.p + 1, sp.ng) + 2 * q1d;
  switch (sp.p) {
    case 1: launch_apply_p<1>(sp, tabB, qd, fq, x, y, st); break;
    case 2: launch_apply_p<2>(sp, tabB, qd, fq, x, y, st); break;
    case 3: launch_apply_p<3>(sp, tabB, qd, fq, x, y, st); break;
    case 4: launch_apply_p<4>(sp, tabB, qd, fq, x, y, st); break;
    case 5: launch_apply_p<5>(sp, tabB, qd, fq, x, y, st); break;
    case 6: launch_apply_p<6>(sp, tabB, qd, fq, x, y, st); break;
    case 7: launch_apply_p<7>(sp, tabB, qd, fq, x, y, st); break;
    case 8: launch_apply_p<8>(sp, tabB, qd, fq, x, y, st); break;
    default: throw Error(PAFEM_EUNSUPPORTED, "DG apply: order not built");
  }
  HIP_LAUNCH_CHECK_DG();
}

}  // namespace pafem
