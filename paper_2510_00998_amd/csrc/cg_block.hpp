// The Q1 V-cycle below a level in one workgroup: every level from lv[0] down
// has at most CG_BLOCK_MAX_VERTICES vertices, one per thread.  Vectors live in
// LDS, a vertex's stencil in the registers of its thread, so that a step costs
// an LDS round trip instead of one through the L2 cache (7^3 vertices, FP32:
// 9.3 us; 13.6 with the vectors and stencils in global memory).  Steps, their order
// and the per-vertex arithmetic are those of the level-by-level launches.
#pragma once
#include "cg_tiles.hpp"

namespace hpmg {
namespace cgb {

constexpr int DENSE_LDS = 1024;  // entries of the coarsest inverse staged in LDS (m <= 32)

template <typename T>
struct Lds {
  double A[DENSE_LDS];
  T b[CG_BLOCK_POOL], u[CG_BLOCK_POOL];  // every level, one after another
  T w[2][CG_BLOCK_MAX_VERTICES];         // iterates of the current level
  T r[CG_BLOCK_MAX_VERTICES];
};

// (A u) at vertex x; neighbour indices clamped into the grid (the stencil
// entry of a neighbour outside the interior is zero).
template <typename T, int D>
__device__ __forceinline__ T stencil_at(const T (&sv)[cgt::nst<D>()], const int (&x)[3], int nv, const T* u) {
  int cx[3], cy[3], cz[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    cx[d] = min(max(x[0] + d - 1, 0), nv - 1);
    cy[d] = min(max(x[1] + d - 1, 0), nv - 1) * nv;
    cz[d] = (D == 3) ? min(max(x[2] + d - 1, 0), nv - 1) * nv * nv : 0;
  }
  T au = 0;
#pragma unroll
  for (int s = 0; s < cgt::nst<D>(); ++s) au += sv[s] * u[cx[s % 3] + cy[(s / 3) % 3] + cz[(D == 3) ? s / 9 : 1]];
  return au;
}

// Args: CGBlockArgs<T>, as a kernel argument or in constant memory.
template <typename T, int D, int RK, typename Args>
__device__ __forceinline__ void vcycle(Args& a, int col, Lds<T>& S) {
  constexpr int NS = cgt::nst<D>();
  const int v = threadIdx.x;
  T sv[NS], dv = 0;
  int x[3] = {0, 0, 0};
  auto load = [&](auto& L) {  // the thread's vertex, stencil and inverse diagonal
    const int w = v < L.size ? v : 0;
    x[0] = w % L.nv;
    x[1] = w / L.nv % L.nv;
    x[2] = D == 3 ? w / (L.nv * L.nv) : 0;
    cgt::load_stencil<T, D>(L.st, L.size, -1, w, sv);
    dv = L.dinv[w];
  };
  load(a.lv[0]);
  const bool lds_inv = a.m * a.m <= DENSE_LDS;
  if (lds_inv)
    for (int i = v; i < a.m * a.m; i += CG_BLOCK_MAX_VERTICES) S.A[i] = a.Ainv[i];
  if (v < a.lv[0].size)
    S.b[v] = a.contrib ? cgt::gather_corners_at<T, D>(x, a.lv[0].nv + 1, a.contrib + (size_t)col * a.scon)
                       : a.lv[0].b[(size_t)col * a.lv[0].size + v];
  int off = 0;
  for (int l = 0; l + 1 < a.nlev; ++l) {
    auto& L = a.lv[l];
    auto& C = a.lv[l + 1];
    if (l > 0) load(L);
    const bool in = v < L.size;
    __syncthreads();  // b of the level
    const T b = in ? S.b[off + v] : T(0);
    T u = 0;
    int c = 0;
    for (int i = 0; i < a.nu_pre; ++i) {
      const T au = i == 0 ? T(0) : stencil_at<T, D>(sv, x, L.nv, S.w[c]);
      u = u + a.omega * dv * (b - au);
      c ^= 1;
      if (in) S.w[c][v] = u;
      __syncthreads();
    }
    if (a.nu_pre == 0) {
      if (in) S.w[c][v] = T(0);
      __syncthreads();
    }
    if (in) {
      S.u[off + v] = u;
      S.r[v] = b - stencil_at<T, D>(sv, x, L.nv, S.w[c]);
    }
    __syncthreads();
    if (v < C.size) {
      const int y[3] = {v % C.nv, v / C.nv % C.nv, D == 3 ? v / (C.nv * C.nv) : 0};
      S.b[off + L.size + v] = cgt::restrict_box<T, D, RK>(cgt::Parents<T, D, RK>(L.ridx, L.rw, y, {0, 0, 0}), {0, 0, 0}, L.nv, S.r);
    }
    off += L.size;
  }
  __syncthreads();
  if (v < a.m) {
    const double* row = (lds_inv ? S.A : a.Ainv) + (size_t)v * a.m;
    double s = 0.0;
    for (int j = 0; j < a.m; ++j) s += row[j] * (double)S.b[off + j];
    S.u[off + v] = (T)s;
    if (a.nlev == 1) a.lv[0].u[(size_t)col * a.lv[0].size + v] = (T)s;
  }
  if (a.m == 0 && v == 0) S.u[off] = T(0);  // a coarsest grid without interior vertices: e_c = 0
  for (int l = a.nlev - 2; l >= 0; --l) {
    auto& L = a.lv[l];
    auto& C = a.lv[l + 1];
    if (a.nlev > 2) load(L);  // else level 0's are still there
    const bool in = v < L.size;
    const int offc = off;
    off -= L.size;
    __syncthreads();  // the coarser level's u
    T u = 0;
    const T b = in ? S.b[off + v] : T(0);
    if (in) {
      u = S.u[off + v];
      u += cgt::prolong_xyz<T, D>(cgt::Parents<T, D, 2>(L.pidx, L.pw, x, {0, 0, 0}), C.nv, S.u + offc);
      S.w[0][v] = u;
    }
    __syncthreads();
    int c = 0;
    for (int i = 0; i < a.nu_post; ++i) {
      const T au = stencil_at<T, D>(sv, x, L.nv, S.w[c]);
      u = u + a.omega * dv * (b - au);
      c ^= 1;
      if (in) S.w[c][v] = u;
      __syncthreads();
    }
    if (in) {
      S.u[off + v] = u;
      if (l == 0) L.u[(size_t)col * L.size + v] = u;
    }
  }
}

}  // namespace cgb
}  // namespace hpmg
