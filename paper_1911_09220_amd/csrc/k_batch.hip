// Batched operator action: many right-hand sides over many meshes.
//
// Each mesh m holds nrhs vectors stored right-hand-side fastest, X_m[dof][rhs],
// so the gather of one dof reads one contiguous run of nrhs values.  The
// partial-assembly stages are those of the single-vector kernel (G, B, D, B^t,
// G^t; "Operator Decomposition"), one 1D line per thread, applied to NRB
// right-hand sides at once: the tile of a workgroup is NE elements x Q*Q lines x
// NRB right-hand sides with the rhs index fastest (coalesced X loads and Y
// atomics, broadcast D loads, conflict-free LDS).  Table entries are the same for
// every lane and come from scalar loads; the quadrature data D goes through LDS or
// is loaded one plane ahead of its use.  One workgroup per tile and chunk of NRB
// right-hand sides (small tiles: per tile and several chunks, mrhs_walks); the chunks of a tile
// follow each other on one die, whose L2 keeps D and the dof map.  All meshes of one order share
// one grouped launch: a workgroup finds its mesh from a prefix table of tile counts.
//
// Bound by latency at the waves that the registers and LDS leave, and by the atomics (an
// interior node's sum is stored, no other element has it; the others are added).  Loads
// return in order, so the dof ids are loaded before D: behind D's loads they, and with them
// X, waited for D (p = 4 241 -> 230 us, p = 2 278 -> 259).  16
// right-hand sides in FP64, best tile, with D and every stage's addresses held in
// registers across a loop over the chunks (180 at p = 4: one workgroup of 5 waves per CU) ->
// now: p = 1 (64^3 elements) 557 -> 369 us, p = 2 (40^3) 368 -> 257, p = 3 (24^3) 263 -> 156,
// p = 4 (20^3) 442 -> 222, p = 5 (15^3) 280 -> 158, p = 6 (12^3) 207 -> 138.
#include <algorithm>
#include <type_traits>

#include "batch.hpp"
#include "device.hpp"

namespace pafem {

namespace {

template <typename TC, typename TD>
struct Pair {
  typedef TD type __attribute__((ext_vector_type(2)));
};

// Waves per SIMD to compile for: what the LDS of the tile allows a CU, at most what the
// z-line's arrays leave registers for.
constexpr int mrhs_waves(int P, int threads, int lds) {
  const int wgs = (160 * 1024) / lds, waves = wgs * ((threads + 63) / 64) / 4;
  const int cap = P <= 1 ? 7 : P <= 3 ? 5 : P <= 5 ? 4 : 3;
  return waves < 1 ? 1 : waves < cap ? waves : cap;
}

// Whether the elements' D goes through LDS: loaded once for the tile, under the latency of X,
// where the streamed variant reads every plane in each right-hand side's thread.  16
// right-hand sides, streamed -> LDS: p = 1 (tile 16, 64^3 elements) 424 -> 354 us, p = 2 (16,
// 40^3) 297 -> 237, p = 3 (16, 24^3) 156 -> 139, p = 4 (4, 20^3) 203 -> 193, p = 5 (8, 15^3) 137.5 ->
// 135; FP32 p = 4 (8) 127 -> 107, p = 5 (8) 95 -> 90.  Tiles of 2 and 4 gain less, as they read D
// fewer times: p = 2 790 -> 737 (2) and 372 -> 340 (4), p = 5 (4) 153 -> 146, but p = 3 301 -> 309 (2)
// and 204 -> 211 (4), p = 5 (2) 207 -> 213, and p = 1 on 56^3 with two right-hand sides 120 -> 129.
// At p = 6 the planes take the LDS of a third workgroup.
constexpr bool mrhs_d_in_lds(int P, int KIND, int NRB, bool f32, bool walk) {
  const bool streamed = (P == 1 && NRB <= 4 && !walk) || ((P == 3 || P == 5) && NRB <= 4);
  return KIND == PAFEM_DIFFUSION && P <= 5 && (f32 || !streamed);
}

// Whether workgroups walk several chunks of right-hand sides, D staying in LDS: tiles of 2 and 4
// at p = 1, 2 and those of 2 at p = 3 in FP32, which are what right-hand sides that 8 does not
// divide get.  Their workgroups are one wave, and with one per chunk the starts of workgroups
// bound the launch.  One workgroup per chunk -> walking: p = 1 on 56^3 elements, 10 right-hand
// sides 679 -> 502 us (FP32 863 -> 501), 14: 909 -> 691 (986 -> 616); on 100^3, 20: 3613 -> 3027
// (3378 -> 2494); p = 2 on 28^3, 10: 200 -> 147 (222 -> 166); on 50^3, 54: 5260 -> 4042 (6866 ->
// 4617); p = 3 on 33^3 in FP32, 14: 826 -> 688, but 775 -> 950 in FP64 (D streamed).  Tiles of 2
// that walk go in launch order, not in die order: p = 1 on 100^3 in FP32, 6: 1841 -> 1624, 54:
// 12923 -> 11630, p = 2 on 50^3, 6: 577 -> 517 (tiles of 4 the other way: p = 1 on 100^3 in FP32,
// 20: 2494 -> 2915).
constexpr bool mrhs_walks(int P, int NRB, bool f32) {
  return (P <= 2 && NRB <= 4) || (P == 3 && NRB == 2 && f32);
}

// The right-hand sides of a launch that does not simply take one workgroup per tile and chunk:
// ngroup groups of `walk` chunks, from first_rhs up to end_rhs.  A type of its own, as one more
// argument in every launch took the scalar registers of an eighth wave at p = 4 in FP32 (16
// right-hand sides on 25^3 elements 217 -> 230 us).
struct RhsPart {
  int ngroup, walk, first_rhs, end_rhs;
};
struct NoPart {};

template <int P, int Q, int NE, int NRB, int KIND, bool PART, typename TV, typename TD, typename TC>
__global__ void __launch_bounds__(
    NE * Q * Q * NRB,
    mrhs_waves(P, NE * Q * Q * NRB,
               NE * Q * Q *
                   ((KIND == PAFEM_DIFFUSION ? 3 : 1) * (P + 1) * NRB * int(sizeof(TC)) +
                    (mrhs_d_in_lds(P, KIND, NRB, sizeof(TC) == 4, PART) ? 6 * Q * int(sizeof(TD))
                                                                       : 0))))
    pa_apply_mrhs_kernel(const BatchMesh* __restrict__ meshes, int nmesh,
                         const TC* __restrict__ tabB, const TC* __restrict__ tabG, int nrhs,
                         std::conditional_t<PART, RhsPart, NoPart> part) {
  constexpr int D = P + 1, DD = D * D, QQ = Q * Q;
  constexpr bool DIFF = (KIND == PAFEM_DIFFUSION);
  constexpr int NC = DIFF ? 6 : 1;
  constexpr int NCC = DIFF ? 3 : 1;
  constexpr int ELEM = NCC * QQ * D;  // entries of one element region (per rhs)
  static_assert((DIFF ? 2 : 1) * D <= NCC * Q, "x-line outputs must fit the element region");

  constexpr bool DLDS = mrhs_d_in_lds(P, KIND, NRB, sizeof(TC) == 4, PART);
  typedef typename Pair<TC, TD>::type pair_t;
  __shared__ TC sW[NE * ELEM * NRB];
  __shared__ pair_t sD[DLDS ? NE * 3 * Q * QQ : 1];  // [el][k, qz][line]

  // which mesh, which tile of it and which right-hand sides.  In die order: consecutive
  // workgroups of one die take the chunks of a tile and then its neighbour, so D, the dof map
  // and the shared dofs' lines stay in that die's L2
  constexpr bool WALK = PART && mrhs_walks(P, NRB, sizeof(TC) == 4);
  int m = 0;
  const int blk = WALK && NRB == 2 ? int(blockIdx.x) : xcd_remap(blockIdx.x, gridDim.x);
  int ngroup = nrhs / NRB;
  if constexpr (PART) ngroup = part.ngroup;
  const int t = blk / ngroup;
  while (m + 1 < nmesh && meshes[m + 1].tile_begin <= t) ++m;
  const BatchMesh& M = meshes[m];
  const int tile = t - M.tile_begin;
  int r0 = (blk - t * ngroup) * NRB, r1 = 0;
  if constexpr (PART) {
    r0 = part.first_rhs + r0 * (WALK ? part.walk : 1);
    r1 = WALK ? min(r0 + part.walk * NRB, part.end_rhs) : 0;
  }

  const int constrained = M.constrained;
  auto bB = [&](int q, int d) -> TC { return tabB[q * D + d]; };
  auto bG = [&](int q, int d) -> TC { return tabG[q * D + d]; };
  const TV* __restrict__ X = static_cast<const TV*>(M.x);
  TV* __restrict__ Y = static_cast<TV*>(M.y);

  const int tid = threadIdx.x;
  const int rb = tid % NRB;
  const int pl = tid / NRB;  // line thread: (el, r)
  const int el = NE == 1 ? 0 : pl / QQ;  // one element: e, and with it D's address, uniform
  const int r = pl - el * QQ;
  const int e = tile * NE + el;
  const bool act = e < M.ne;
  TC* const W = sW + el * ELEM * NRB + rb;
  // entry (c, qy, qx, dz) of this element and rhs; the x-line outputs (a, dz, dy, qx)
  // live at c*Q + qy = a*D + dy
  auto at = [&](int c, int qy, int qx, int dz) -> TC& {
    return W[(((c * Q + qy) * Q + qx) * D + dz) * NRB];
  };
  // D of this thread's z-line (qy, qx) = r, a plane at a time: all of it held in
  // registers (12 Q of them) left one workgroup of 5 waves per CU at p = 4
  constexpr int NT = qdata_tile(Q), PL = NT * QQ;  // elements of a qdata tile, values a plane
  const TD* const qe = static_cast<const TD*>(M.qdata) + size_t(e / NT) * (NC * Q * PL) +
                       (DIFF ? 2 : 1) * ((e % NT) * QQ);
  const unsigned rq = (DIFF ? 2 : 1) * r;
  TC dq[Q][NC];
  auto load_plane = [&](int qz) {
    if constexpr (DIFF) {
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        pair_t v;
        if constexpr (DLDS)
          v = sD[(el * 3 * Q + k * Q + qz) * QQ + r];
        else
          v = *reinterpret_cast<const pair_t*>(qe + 2 * ((k * Q + qz) * PL) + rq);
        dq[qz][2 * k] = TC(v.x);
        dq[qz][2 * k + 1] = TC(v.y);
      }
    } else {
      dq[qz][0] = TC(qe[qz * PL + rq]);
    }
  };
  // x-line (dz, dy) = r < D*D: the dofs of its D nodes, read again before the scatter
  const bool xline = act && r < DD;
  const int xz = r / D, xy = r - (r / D) * D;
  const bool xline_inner = xz > 0 && xz < P && xy > 0 && xy < P;
  const int32_t* __restrict__ gline = M.gmap + size_t(e) * (DD * D) + r * D;
  bool first = true;
  do {
  // loads return in order: the dofs first, X waits for nothing else
  int gx[D];
  if (xline) {
#pragma unroll
    for (int dx = 0; dx < D; ++dx) gx[dx] = gline[dx];
  }
  // DLDS: row j = (k, qz) of the line is loaded by the thread of right-hand side j mod NRB,
  // under the first contraction's loads
  constexpr int NJ = DLDS ? (3 * Q + NRB - 1) / NRB : 1;
  pair_t dj[NJ];
  if constexpr (DLDS) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (act && first && rb + j * NRB < 3 * Q)
        dj[j] = *reinterpret_cast<const pair_t*>(qe + size_t(2 * PL) * (rb + j * NRB) + rq);
  }
  const bool yline = act && r < D * Q;
  const int yz = r / Q, yx = r - (r / Q) * Q;
  const int zy = r / Q, zx = r - (r / Q) * Q;
  const int rr = r0 + rb;
  // G and B along x: thread (dz, dy)
  if (xline) {
    TC u[D];
#pragma unroll
    for (int dx = 0; dx < D; ++dx) {
      const int g = gx[dx];
      u[dx] = (constrained && g < 0) ? TC(0) : TC(X[size_t(g < 0 ? ~g : g) * nrhs + rr]);
    }
#pragma unroll
    for (int qx = 0; qx < Q; ++qx) {
      TC b = TC(0), g = TC(0);
#pragma unroll
      for (int dx = 0; dx < D; ++dx) {
        b += bB(qx, dx) * u[dx];
        if (DIFF) g += bG(qx, dx) * u[dx];
      }
      at(xy / Q, xy % Q, qx, xz) = b;
      if (DIFF) at((D + xy) / Q, (D + xy) % Q, qx, xz) = g;
    }
  }
  if constexpr (DLDS) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      if (act && first && rb + j * NRB < 3 * Q) sD[(el * 3 * Q + rb + j * NRB) * QQ + r] = dj[j];
  }
  __syncthreads();
  // B along y: thread (dz, qx)
  if (yline) {
    TC aB[D], aG[D];
#pragma unroll
    for (int dy = 0; dy < D; ++dy) {
      aB[dy] = at(dy / Q, dy % Q, yx, yz);
      if (DIFF) aG[dy] = at((D + dy) / Q, (D + dy) % Q, yx, yz);
    }
#pragma unroll
    for (int qy = 0; qy < Q; ++qy) {
      TC gb = TC(0), bg = TC(0), bb = TC(0);
#pragma unroll
      for (int dy = 0; dy < D; ++dy) {
        bb += bB(qy, dy) * aB[dy];
        if (DIFF) {
          gb += bB(qy, dy) * aG[dy];
          bg += bG(qy, dy) * aB[dy];
        }
      }
      if (DIFF) {
        at(0, qy, yx, yz) = gb;
        at(1, qy, yx, yz) = bg;
        at(2, qy, yx, yz) = bb;
      } else {
        at(0, qy, yx, yz) = bb;
      }
    }
  }
  __syncthreads();
  // B along z, D, B^t along z: thread (qy, qx), in place
  if (act) {
    load_plane(0);
    TC c0[D], c1[D], c2[D];
#pragma unroll
    for (int dz = 0; dz < D; ++dz) {
      c0[dz] = at(0, zy, zx, dz);
      if (DIFF) {
        c1[dz] = at(1, zy, zx, dz);
        c2[dz] = at(2, zy, zx, dz);
      }
    }
    TC t0[D], t1[D], t2[D];
#pragma unroll
    for (int dz = 0; dz < D; ++dz) t0[dz] = t1[dz] = t2[dz] = TC(0);
#pragma unroll
    for (int qz = 0; qz < Q; ++qz) {
      if (DLDS && qz > 0) load_plane(qz);
      if (!DLDS && qz + 1 < Q) load_plane(qz + 1);
      __asm__ volatile("" ::: "memory");  // keep the next plane's loads in this iteration
      if (DIFF) {
        TC ux = TC(0), uy = TC(0), uz = TC(0);
#pragma unroll
        for (int dz = 0; dz < D; ++dz) {
          ux += bB(qz, dz) * c0[dz];
          uy += bB(qz, dz) * c1[dz];
          uz += bG(qz, dz) * c2[dz];
        }
        const TC vx = dq[qz][0] * ux + dq[qz][1] * uy + dq[qz][2] * uz;
        const TC vy = dq[qz][1] * ux + dq[qz][3] * uy + dq[qz][4] * uz;
        const TC vz = dq[qz][2] * ux + dq[qz][4] * uy + dq[qz][5] * uz;
#pragma unroll
        for (int dz = 0; dz < D; ++dz) {
          t0[dz] += bB(qz, dz) * vx;
          t1[dz] += bB(qz, dz) * vy;
          t2[dz] += bG(qz, dz) * vz;
        }
      } else {
        TC u = TC(0);
#pragma unroll
        for (int dz = 0; dz < D; ++dz) u += bB(qz, dz) * c0[dz];
        const TC v = dq[qz][0] * u;
#pragma unroll
        for (int dz = 0; dz < D; ++dz) t0[dz] += bB(qz, dz) * v;
      }
    }
#pragma unroll
    for (int dz = 0; dz < D; ++dz) {
      at(0, zy, zx, dz) = t0[dz];
      if (DIFF) {
        at(1, zy, zx, dz) = t1[dz];
        at(2, zy, zx, dz) = t2[dz];
      }
    }
  }
  __syncthreads();
  // B^t along y: thread (dz, qx)
  if (yline) {
    TC v0[Q], v1[Q], v2[Q];
#pragma unroll
    for (int qy = 0; qy < Q; ++qy) {
      v0[qy] = at(0, qy, yx, yz);
      if (DIFF) {
        v1[qy] = at(1, qy, yx, yz);
        v2[qy] = at(2, qy, yx, yz);
      }
    }
#pragma unroll
    for (int dy = 0; dy < D; ++dy) {
      TC b = TC(0), g = TC(0);
#pragma unroll
      for (int qy = 0; qy < Q; ++qy) {
        if (DIFF) {
          g += bB(qy, dy) * v0[qy];
          b += bG(qy, dy) * v1[qy] + bB(qy, dy) * v2[qy];
        } else {
          b += bB(qy, dy) * v0[qy];
        }
      }
      at(dy / Q, dy % Q, yx, yz) = b;
      if (DIFF) at((D + dy) / Q, (D + dy) % Q, yx, yz) = g;
    }
  }
  if (xline) {
#pragma unroll
    for (int dx = 0; dx < D; ++dx) gx[dx] = gline[dx];
  }
  __syncthreads();
  // B^t along x and G^t: thread (dz, dy)
  if (xline) {
    TC wB[Q], wG[Q];
#pragma unroll
    for (int qx = 0; qx < Q; ++qx) {
      wB[qx] = at(xy / Q, xy % Q, qx, xz);
      if (DIFF) wG[qx] = at((D + xy) / Q, (D + xy) % Q, qx, xz);
    }
#pragma unroll
    for (int dx = 0; dx < D; ++dx) {
      TC acc = TC(0);
#pragma unroll
      for (int qx = 0; qx < Q; ++qx) {
        acc += bB(qx, dx) * wB[qx];
        if (DIFF) acc += bG(qx, dx) * wG[qx];
      }
      const int g = gx[dx];
      TV* const dst = &Y[size_t(g < 0 ? ~g : g) * nrhs + rr];
      if (dx > 0 && dx < P && xline_inner)  // an interior node: no other element has it
        *dst = TV(acc);
      else if (!(constrained && g < 0))
        unsafeAtomicAdd(dst, TV(acc));
    }
  }
  if constexpr (WALK) {
    first = false;
    r0 += NRB;
    if (r0 < r1) __syncthreads();  // the next chunk overwrites the element regions
  }
  } while (WALK && r0 < r1);
}

// Y = X on essential dofs (constrained) and 0 elsewhere, for every mesh of the
// batch; blockIdx.y selects the mesh.  nrhs is even: a thread sets two right-hand sides
// of a dof, and divides once instead of once per value.
template <typename TV>
__global__ void __launch_bounds__(256)
    batch_init_kernel(const BatchMesh* __restrict__ meshes, int nrhs) {
  const BatchMesh& M = meshes[blockIdx.y];
  const int pairs = nrhs / 2;
  const int rows = pairs < 256 ? 256 / pairs : 1;  // dofs of a workgroup
  const int row = int(threadIdx.x) / pairs, p0 = int(threadIdx.x) - row * pairs;
  if (pairs < 256 && row >= rows) return;
  const TV* __restrict__ X = static_cast<const TV*>(M.x);
  TV* __restrict__ Y = static_cast<TV*>(M.y);
  for (int64_t g = int64_t(blockIdx.x) * rows + (pairs < 256 ? row : 0); g < M.ndofs;
       g += int64_t(gridDim.x) * rows) {
    const bool keep = M.constrained && M.bmask[g];
    for (int p = pairs < 256 ? p0 : int(threadIdx.x); p < pairs; p += 256) {
      const int64_t k = g * nrhs + 2 * p;
      const TV a = keep ? X[k] : TV(0), b = keep ? X[k + 1] : TV(0);
      Y[k] = a;
      Y[k + 1] = b;
    }
  }
}

// Walking workgroups take all right-hand sides of a tile from this many tiles on; fewer tiles are
// split into groups of chunks that make up for it (54 right-hand sides, all at once -> grouped:
// p = 2 on 8^3 elements 67 -> 30 us, on 12^3 86 -> 74, p = 1 on 8^3 54 -> 26; on 16^3, 4096 tiles,
// 138 and 77 where 8 groups took 144 and 78)
constexpr int64_t kWalkTiles = 4096;

template <int P, int NE, int NRB, typename TV, typename TD, typename TC>
void launch_cfg(const BatchMesh* meshes, int nmesh, int64_t ntiles, int kind, const void* tab,
                int nrhs, hipStream_t st) {
  constexpr int Q = P + 2, T = NE * Q * Q * NRB;
  const int chunks = nrhs / NRB;
  // groups of chunks, one workgroup each: as even as possible
  int groups = chunks;
  if (mrhs_walks(P, NRB, sizeof(TC) == 4))
    groups = int(std::min<int64_t>(chunks, (kWalkTiles + ntiles - 1) / ntiles));
  const int walk = (chunks + groups - 1) / groups;
  groups = (chunks + walk - 1) / walk;
  const int per = batch_launch_groups(ntiles, T, groups);
  const TC* tabB = static_cast<const TC*>(tab);
  const TC* tabG = tabB + Q * (P + 1);
  for (int g = 0; g < groups; g += per) {
    const int ng = std::min(per, groups - g);
    const dim3 grid(unsigned(ntiles * ng));
    auto launch = [&](auto kernel, auto part) {
      hipLaunchKernelGGL(kernel, grid, dim3(T), 0, st, meshes, nmesh, tabB, tabG, nrhs, part);
    };
    auto launch_kind = [&](auto part) {
      constexpr bool PART = !std::is_same<decltype(part), NoPart>::value;
      if (kind == PAFEM_DIFFUSION)
        launch(pa_apply_mrhs_kernel<P, Q, NE, NRB, PAFEM_DIFFUSION, PART, TV, TD, TC>, part);
      else
        launch(pa_apply_mrhs_kernel<P, Q, NE, NRB, PAFEM_MASS, PART, TV, TD, TC>, part);
    };
    if (walk > 1 || ng < chunks)
      launch_kind(RhsPart{ng, walk, g * walk * NRB, nrhs});
    else
      launch_kind(NoPart{});
  }
}

// Candidate tiles per order (elements x right-hand sides per workgroup), limited
// by 1024 threads per workgroup and the LDS of the FP64 diffusion variant.
template <int P, typename TV, typename TD, typename TC>
bool launch_tile(int cand, const BatchMesh* meshes, int nmesh, int64_t ntiles, int kind,
                 const void* tab, int nrhs, hipStream_t st) {
  if (cand == 0) {
    launch_cfg<P, 1, 4, TV, TD, TC>(meshes, nmesh, ntiles, kind, tab, nrhs, st);
    return true;
  }
  if (cand == 4) {
    launch_cfg<P, 1, 2, TV, TD, TC>(meshes, nmesh, ntiles, kind, tab, nrhs, st);
    return true;
  }
  if constexpr (P <= 5) {
    if (cand == 1) {
      launch_cfg<P, 1, 8, TV, TD, TC>(meshes, nmesh, ntiles, kind, tab, nrhs, st);
      return true;
    }
  }
  if constexpr (P <= 3) {
    if (cand == 2) {
      launch_cfg<P, 1, 16, TV, TD, TC>(meshes, nmesh, ntiles, kind, tab, nrhs, st);
      return true;
    }
  }
  if constexpr (P <= 3) {
    if (cand == 3) {
      launch_cfg<P, 2, 8, TV, TD, TC>(meshes, nmesh, ntiles, kind, tab, nrhs, st);
      return true;
    }
  }
  return false;
}

}  // namespace

int batch_tile_elems(int cand) {
  switch (cand) {
    case 3: return 2;
    default: return 1;
  }
}
int batch_tile_rhs(int cand) {
  switch (cand) {
    case 0: return 4;
    case 1: return 8;
    case 2: return 16;
    case 3: return 8;
    case 4: return 2;
    case kBatchMfmaCandidate: return 16;
    default: return 0;
  }
}

bool launch_batch_apply(int p, int cand, int vdtype, int qdtype, int kind,
                        const BatchMesh* meshes, int nmesh, int64_t ntiles, const void* tab,
                        int nrhs, hipStream_t st) {
  if (cand == kBatchMfmaCandidate) {
    if (vdtype != PAFEM_F64 || qdtype != PAFEM_F64 || nrhs % 16) return false;
    return launch_batch_apply_mfma(p, kind, meshes, nmesh, int(ntiles),
                                   static_cast<const double*>(tab), nrhs, st);
  }
  bool ok = false;
#define PAFEM_BATCH_ORDER(PP)                                                                   \
  case PP:                                                                                      \
    if (vdtype == PAFEM_F64 && qdtype == PAFEM_F64)                                             \
      ok = launch_tile<PP, double, double, double>(cand, meshes, nmesh, ntiles, kind, tab,     \
                                                   nrhs, st);                                   \
    else if (vdtype == PAFEM_F32 && qdtype == PAFEM_F32)                                        \
      ok = launch_tile<PP, float, float, float>(cand, meshes, nmesh, ntiles, kind, tab, nrhs,  \
                                                st);                                            \
    break;
  switch (p) {
    PAFEM_BATCH_ORDER(1)
    PAFEM_BATCH_ORDER(2)
    PAFEM_BATCH_ORDER(3)
    PAFEM_BATCH_ORDER(4)
    PAFEM_BATCH_ORDER(5)
    PAFEM_BATCH_ORDER(6)
    default: ok = false;
  }
#undef PAFEM_BATCH_ORDER
  if (ok) {
    hipError_t err = hipGetLastError();
    if (err != hipSuccess)
      throw Error(PAFEM_EHIP, std::string("batch apply launch: ") + hipGetErrorString(err));
  }
  return ok;
}

void launch_batch_init(int vdtype, const BatchMesh* meshes, int nmesh, int nrhs,
                       hipStream_t st) {
  const dim3 grid(1024, unsigned(nmesh));
  if (vdtype == PAFEM_F64)
    hipLaunchKernelGGL(batch_init_kernel<double>, grid, dim3(256), 0, st, meshes, nrhs);
  else
    hipLaunchKernelGGL(batch_init_kernel<float>, grid, dim3(256), 0, st, meshes, nrhs);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess)
    throw Error(PAFEM_EHIP, std::string("batch init launch: ") + hipGetErrorString(err));
}

}  // namespace pafem
