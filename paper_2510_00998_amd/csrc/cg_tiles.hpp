// Q1 levels in tiles: one workgroup carries a tile of a level through several
// steps of the cycle in LDS, recomputing the values its neighbours also need,
// so that a level takes one launch on the way down (all pre-smoothing steps
// from zero, the residual, its restriction) and one on the way up (the
// prolongation, all post-smoothing steps).
//
// Bound: latency.  The levels hold at most some 10^5 vertices, a launch of
// one step takes about 4 us whatever it does, and a cycle had 3 launches up
// and 4 or 5 down per level.  The steps of a tile share one read of each
// vertex's stencil, kept in registers, or take it from scalar loads where all
// vertices have the same.  31^3 and 15^3 vertices in FP32 with two steps each
// way: 8 launches of 3.3 to 4.3 us down to one of 8.3 us on the way down (11.2
// with a stencil per vertex), 3 to one of 5.6 us on the way up (7.2).  A small
// tile, 2 coarse vertices per axis in 3D, suits one problem: with 4 the
// recomputed share falls from 5.4 to 2.6 times the tile, but 64 workgroups
// leave most of the chip idle (15.4 against 11.2 us).  Per-vertex arithmetic
// and its order are those of the single-step kernels (cg_stencil_at,
// restrict_box, prolong_xyz), so the results are the same bit for bit.
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace hpmg {
namespace cgt {

constexpr int cpow(int b, int e) { return e == 0 ? 1 : b * cpow(b, e - 1); }

// Tile of a level: CT coarse vertices per axis on the way down, FT fine
// vertices on the way up; RK = 2 factor - 1 fine vertices per coarse one.
template <int D, int RK, int CTILE>
struct Tile {
  static constexpr int HF = (RK + 1) / 2;
  static constexpr int CT = CTILE, FT = HF * CT;
  static constexpr int ER = HF * CT + HF - 1;  // extent of the residual's box
  static constexpr int EM = 2;                 // largest smoothing count
  static constexpr int EB = ER + 2 * EM, EU = ER + 2 * (EM - 1);
  static constexpr int NB = cpow(EB, D), NU = cpow(EU, D), NR = cpow(ER, D), NC = cpow(CT, D);
  // every step takes at most two rounds of the workgroup (its stencils stay in
  // registers)
  static constexpr int THREADS = (NU / 2 + 255) / 256 * 256;
  static_assert(NC <= THREADS, "one coarse vertex per thread");
  static constexpr int RPT = (NU + THREADS - 1) / THREADS;
  template <typename T>
  static constexpr int lds_bytes() {
    return (int)sizeof(T) * (2 * NB + NU + NR);
  }
};

template <int D>
constexpr int nst() {
  return D == 2 ? 9 : 27;
}

// Fine interior indices and weights of a coarse vertex along one axis
// (RK slots; an empty slot, index < 0, becomes index `none` with weight 0).
template <typename T, int RK>
__device__ __forceinline__ void axis_parents(const int* __restrict__ idx, const T* __restrict__ w, int x, int none,
                                             int (&i)[RK], T (&wt)[RK]) {
#pragma unroll
  for (int a = 0; a < RK; ++a) {
    const int k = idx[RK * x + a];
    i[a] = k < 0 ? none : k;
    wt[a] = k < 0 ? T(0) : w[RK * x + a];
  }
}

// Transfer entries of one vertex along every axis, loaded ahead of their use.
template <typename T, int D, int RK>
struct Parents {
  int i[3][RK];
  T w[3][RK];
  __device__ __forceinline__ Parents(const int* __restrict__ idx, const T* __restrict__ wt, const int (&x)[3],
                                     const int (&none)[3]) {
#pragma unroll
    for (int k = 0; k < D; ++k) axis_parents<T, RK>(idx, wt, x[k], none[k], i[k], w[k]);
  }
};

// (P^T r_f) at a coarse interior vertex with the tensor-product 1D transfer:
// up to RK = 2f - 1 fine interior indices per axis (f = 2 or 3: the coarsening
// factor).  r_f on a box with origin lo and rows of E entries (the whole
// level: origin 0, E = its extent).
template <typename T, int D, int RK>
__device__ __forceinline__ T restrict_box(const Parents<T, D, RK>& P, const int (&lo)[3], int E, const T* rf) {
  T s = 0;
#pragma unroll
  for (int c = 0; c < (D == 3 ? RK : 1); ++c)
#pragma unroll
    for (int b2 = 0; b2 < RK; ++b2)
#pragma unroll
      for (int a2 = 0; a2 < RK; ++a2)
        s += (D == 3 ? P.w[2][c] : T(1)) * P.w[1][b2] * P.w[0][a2] *
             rf[P.i[0][a2] - lo[0] + E * (P.i[1][b2] - lo[1] + (D == 3 ? E * (P.i[2][c] - lo[2]) : 0))];
  return s;
}

// (P e_c) at a fine interior vertex: up to two coarse interior indices per axis.
template <typename T, int D>
__device__ __forceinline__ T prolong_xyz(const Parents<T, D, 2>& P, int nvc, const T* ec) {
  T s = 0;
#pragma unroll
  for (int c = 0; c < (D == 3 ? 2 : 1); ++c)
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
      for (int a2 = 0; a2 < 2; ++a2)
        s += (D == 3 ? P.w[2][c] : T(1)) * P.w[1][b2] * P.w[0][a2] *
             ec[P.i[0][a2] + nvc * (P.i[1][b2] + (D == 3 ? nvc * P.i[2][c] : 0))];
  return s;
}

// Q1 right-hand side at interior vertex x from the corner contributions of
// the restricted DG residual: the sum over the 2^d cells around it.
template <typename T, int D>
__device__ __forceinline__ T gather_corners_at(const int (&x)[3], int n, const T* __restrict__ contrib) {
  constexpr int NCOR = 1 << D;
  T s = 0;
#pragma unroll
  for (int c = 0; c < NCOR; ++c) {
    const int ix = c & 1, iy = (c >> 1) & 1, iz = (c >> 2) & 1;
    const int cx = x[0] + ix, cy = x[1] + iy, cz = (D == 3) ? x[2] + iz : 0;  // vertex v+1 -> cell v+ix
    const int cell = cx + n * (cy + n * cz);
    const int corner = (1 - ix) + 2 * (1 - iy) + ((D == 3) ? 4 * (1 - iz) : 0);
    s += contrib[(size_t)cell * NCOR + corner];
  }
  return s;
}

// Box of extent E per axis: i-th point's offsets.
template <int D, int E>
__device__ __forceinline__ void unpack(int i, int (&x)[3]) {
  x[0] = i % E;
  x[1] = i / E % E;
  x[2] = D == 3 ? i / (E * E) : 0;
}

// Stencil of vertex v into registers.  uni >= 0: every vertex has that
// vertex's stencil (but for the neighbours outside the interior, whose values
// in a box are zero), which comes by scalar loads.
template <typename T, int D>
__device__ __forceinline__ void load_stencil(const T* __restrict__ st, int total, int uni, int v,
                                             T (&sv)[nst<D>()]) {
  if (uni >= 0) {
#pragma unroll
    for (int s = 0; s < nst<D>(); ++s) sv[s] = st[(size_t)s * total + uni];
  } else {
#pragma unroll
    for (int s = 0; s < nst<D>(); ++s) sv[s] = st[(size_t)s * total + v];
  }
}

// (A u) at the box point with array index `at` (extent E).
template <typename T, int D, int E>
__device__ __forceinline__ T stencil_box(const T (&sv)[nst<D>()], const T* u, int at) {
  T au = 0;
#pragma unroll
  for (int s = 0; s < nst<D>(); ++s)
    au += sv[s] * u[at + s % 3 - 1 + E * ((s / 3) % 3 - 1) + (D == 3 ? E * E * (s / 9 - 1) : 0)];
  return au;
}

// Down: b of the tile's surroundings (from memory, or gathered from the DG
// cells' corner contributions and stored), NU Jacobi steps from zero, the
// residual, its restriction to the CT^D coarse vertices of the tile.  u and b
// are stored for the vertices the tile owns.
template <typename T, int D, int RK, int CT, int NU>
__device__ __forceinline__ void down_tile(const CGTileArgs<T>& a, int tile, int rhs, char* lds) {
  using Ti = Tile<D, RK, CT>;
  constexpr int NS = nst<D>(), HF = Ti::HF, EB = Ti::EB, EU = Ti::EU, ER = Ti::ER;
  T* sB = (T*)lds;          // right-hand side, box of the residual grown by NU
  T* sU = sB + Ti::NB;      // first iterate on the same box
  T* sV = sU + Ti::NB;      // second iterate, box grown by one
  T* sR = sV + Ti::NU;      // residual
  const int nv = a.nv, total = D == 2 ? nv * nv : nv * nv * nv;
  const int tx = (a.nvc + Ti::CT - 1) / Ti::CT;
  int t[3] = {tile % tx, tile / tx % tx, D == 3 ? tile / (tx * tx) : 0};
  int I0[3], lo[3], hi[3], olo[3], ohi[3];  // coarse start, residual's box, owned vertices
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (k >= D) {
      I0[k] = lo[k] = hi[k] = olo[k] = ohi[k] = 0;
      continue;
    }
    I0[k] = t[k] * Ti::CT;
    const int I1 = min(I0[k] + Ti::CT, a.nvc);
    lo[k] = HF * I0[k];
    hi[k] = min(nv - 1, HF * (I1 + 1) - 2);
    olo[k] = t[k] == 0 ? 0 : HF * (I0[k] + 1) - 1;
    ohi[k] = I1 == a.nvc ? nv - 1 : HF * (I1 + 1) - 2;
  }
  const T* bin = a.b + (size_t)rhs * a.sf;
  T* bout = const_cast<T*>(bin);
  T* uo = a.u_out + (size_t)rhs * a.sf;
  const T* con = a.contrib ? a.contrib + (size_t)rhs * a.scon : nullptr;
  // stencils of the box grown by NU - 1, loaded first
  T sv[Ti::RPT][NS], dv[Ti::RPT];
  int vv[Ti::RPT];
#pragma unroll
  for (int m = 0; m < Ti::RPT; ++m) {
    int x[3];
    const int i = threadIdx.x + m * Ti::THREADS;
    unpack<D, EU>(i, x);
    bool in = i < Ti::NU;
    int v = 0;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
      const int g = lo[k] - (NU - 1) + x[k];
      in = in && g >= 0 && g < nv && g <= hi[k] + NU - 1;
      v = v * nv + g;
    }
    vv[m] = in ? v : -1;
    load_stencil<T, D>(a.st, total, a.uni, in ? v : 0, sv[m]);
    if (NU == 2) dv[m] = a.uni >= 0 ? a.dinv[a.uni] : a.dinv[in ? v : 0];
  }
  // b and the first step from zero (indices clamped, not branched around, so
  // that every load of the tile is in flight at once)
  constexpr int RB = (Ti::NB + Ti::THREADS - 1) / Ti::THREADS;
  T bb[RB], db[RB];
  int vb[RB];
  bool ownb[RB];
#pragma unroll
  for (int m = 0; m < RB; ++m) {
    int x[3];
    const int i = threadIdx.x + m * Ti::THREADS;
    unpack<D, EB>(i, x);
    bool in = i < Ti::NB;
    ownb[m] = true;
    int g[3] = {0, 0, 0}, v = 0;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
      g[k] = lo[k] - NU + x[k];
      in = in && g[k] >= 0 && g[k] < nv && g[k] <= hi[k] + NU;
      ownb[m] = ownb[m] && g[k] >= olo[k] && g[k] <= ohi[k];
      g[k] = min(max(g[k], 0), nv - 1);
      v = v * nv + g[k];
    }
    vb[m] = in ? v : -1;
    bb[m] = con ? gather_corners_at<T, D>(g, a.n, con) : bin[v];
    db[m] = a.uni >= 0 ? a.dinv[a.uni] : a.dinv[v];
  }
  const int nc0 = threadIdx.x < Ti::NC ? (int)threadIdx.x : 0;
  int I[3];
  unpack<D, Ti::CT>(nc0, I);
  bool inc = threadIdx.x < Ti::NC;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    I[k] += I0[k];
    inc = inc && I[k] < a.nvc;
    I[k] = min(I[k], a.nvc - 1);
  }
  const Parents<T, D, RK> P(a.ridx, a.rw, I, lo);
#pragma unroll
  for (int m = 0; m < RB; ++m) {
    const int i = threadIdx.x + m * Ti::THREADS;
    if (i >= Ti::NB) continue;
    T b = 0, u = 0;
    if (vb[m] >= 0) {
      b = bb[m];
      u = T(0) + a.omega * db[m] * (b - T(0));
      if (ownb[m]) {
        if (con) bout[vb[m]] = b;
        if (NU == 1) uo[vb[m]] = u;
      }
    }
    sB[i] = b;
    sU[i] = u;
  }
  __syncthreads();
  // index in the EB box of point x of a box grown by G
  auto at_b = [&](const int (&x)[3], int G) {
    return x[0] + NU - G + EB * (x[1] + NU - G + (D == 3 ? EB * (x[2] + NU - G) : 0));
  };
  if constexpr (NU == 2) {
#pragma unroll
    for (int m = 0; m < Ti::RPT; ++m) {
      const int i = threadIdx.x + m * Ti::THREADS;
      if (i >= Ti::NU) continue;
      int x[3];
      unpack<D, EU>(i, x);
      T u = 0;
      if (vv[m] >= 0) {
        const int at = at_b(x, 1);
        const T au = stencil_box<T, D, EB>(sv[m], sU, at);
        u = sU[at] + a.omega * dv[m] * (sB[at] - au);
        bool own = true;
#pragma unroll
        for (int k = 0; k < D; ++k) {
          const int g = lo[k] - 1 + x[k];
          own = own && g >= olo[k] && g <= ohi[k];
        }
        if (own) uo[vv[m]] = u;
      }
      sV[i] = u;
    }
    __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < Ti::RPT; ++m) {
    const int i = threadIdx.x + m * Ti::THREADS;
    int x[3];
    unpack<D, EU>(i, x);
    bool inr = vv[m] >= 0;
    int ri = 0;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
      const int y = x[k] - (NU - 1);
      inr = inr && y >= 0 && y < ER && lo[k] + y <= hi[k];
      ri = ri * ER + y;
    }
    if (!inr) continue;
    const int at = at_b(x, NU - 1);
    const T au = NU == 2 ? stencil_box<T, D, EU>(sv[m], sV, i) : stencil_box<T, D, EB>(sv[m], sU, at);
    sR[ri] = sB[at] - au;
  }
  __syncthreads();
  T* bc = a.bc + (size_t)rhs * a.sc;
  if (inc) bc[I[0] + a.nvc * (I[1] + (D == 3 ? a.nvc * I[2] : 0))] = restrict_box<T, D, RK>(P, lo, ER, sR);
}

// Up: u + P e of the tile's surroundings, NU Jacobi steps, stored (into the
// other iterate: neighbouring tiles still read this one).
template <typename T, int D, int RK, int CT, int NU>
__device__ __forceinline__ void up_tile(const CGTileArgs<T>& a, int tile, int rhs, char* lds) {
  using Ti = Tile<D, RK, CT>;
  constexpr int NS = nst<D>(), FT = Ti::FT, EW = FT + 2 * NU, E1 = FT + 2 * (NU - 1);
  constexpr int NW = cpow(EW, D), N1 = cpow(E1, D);
  constexpr int RPT = (N1 + Ti::THREADS - 1) / Ti::THREADS;
  static_assert(NW <= Ti::NB && N1 <= Ti::NU, "fits the boxes of the way down");
  T* sU = (T*)lds;
  T* sV = sU + 2 * Ti::NB;
  const int nv = a.nv, total = D == 2 ? nv * nv : nv * nv * nv;
  const int tx = (nv + FT - 1) / FT;
  const int o[3] = {tile % tx * FT, tile / tx % tx * FT, D == 3 ? tile / (tx * tx) * FT : 0};
  const T* ui = a.u_in + (size_t)rhs * a.sf;
  const T* b = a.b + (size_t)rhs * a.sf;
  const T* ec = a.ec + (size_t)rhs * a.sc;
  T* uo = a.u_out + (size_t)rhs * a.sf;
  T sv[RPT][NS], bv[RPT], dv[RPT];
  int vv[RPT];
#pragma unroll
  for (int m = 0; m < RPT; ++m) {
    int x[3];
    const int i = threadIdx.x + m * Ti::THREADS;
    unpack<D, E1>(i, x);
    bool in = i < N1;
    int v = 0;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
      const int g = o[k] - (NU - 1) + x[k];
      in = in && g >= 0 && g < nv;
      v = v * nv + g;
    }
    vv[m] = in ? v : -1;
    load_stencil<T, D>(a.st, total, a.uni, in ? v : 0, sv[m]);
    bv[m] = b[in ? v : 0];
    dv[m] = a.uni >= 0 ? a.dinv[a.uni] : a.dinv[in ? v : 0];
  }
#pragma unroll
  for (int m = 0; m < (NW + Ti::THREADS - 1) / Ti::THREADS; ++m) {
    int x[3];
    const int i = threadIdx.x + m * Ti::THREADS;
    unpack<D, EW>(i, x);
    bool in = true;
    int g[3] = {0, 0, 0}, v = 0;
#pragma unroll
    for (int k = D - 1; k >= 0; --k) {
      g[k] = o[k] - NU + x[k];
      in = in && g[k] >= 0 && g[k] < nv;
      g[k] = min(max(g[k], 0), nv - 1);
      v = v * nv + g[k];
    }
    T u = ui[v];
    u += prolong_xyz<T, D>(Parents<T, D, 2>(a.pidx, a.pw, g, {0, 0, 0}), a.nvc, ec);
    if (i < NW) sU[i] = in ? u : T(0);
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < RPT; ++m) {
    const int i = threadIdx.x + m * Ti::THREADS;
    if (i >= N1) continue;
    int x[3];
    unpack<D, E1>(i, x);
    T u = 0;
    if (vv[m] >= 0) {
      const int at = x[0] + 1 + EW * (x[1] + 1 + (D == 3 ? EW * (x[2] + 1) : 0));
      const T au = stencil_box<T, D, EW>(sv[m], sU, at);
      u = sU[at] + a.omega * dv[m] * (bv[m] - au);
      if (NU == 1) uo[vv[m]] = u;
    }
    if constexpr (NU == 2) sV[i] = u;
  }
  if constexpr (NU == 2) {
    __syncthreads();
#pragma unroll
    for (int m = 0; m < RPT; ++m) {
      const int i = threadIdx.x + m * Ti::THREADS;
      int x[3];
      unpack<D, E1>(i, x);
      bool own = vv[m] >= 0;
#pragma unroll
      for (int k = 0; k < D; ++k) own = own && x[k] >= 1 && x[k] <= FT;
      if (!own) continue;
      const T au = stencil_box<T, D, E1>(sv[m], sV, i);
      uo[vv[m]] = sV[i] + a.omega * dv[m] * (bv[m] - au);
    }
  }
}

// Tiles of a level on the way down / up.
template <int D, int CT>
inline int down_tiles(int nvc) {
  return cpow((nvc + CT - 1) / CT, D);
}
template <int D, int RK, int CT>
inline int up_tiles(int nv) {
  constexpr int FT = Tile<D, RK, CT>::FT;
  return cpow((nv + FT - 1) / FT, D);
}

}  // namespace cgt
}  // namespace hpmg
