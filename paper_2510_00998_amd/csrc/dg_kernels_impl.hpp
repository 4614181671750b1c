// Kernel bodies for dg_kernels.hpp (included by the per-instantiation .hip
// files).  See dg_kernels.hpp for the mathematics.
//
// Every thread owns the line of a cell along the last axis (z in 3D): its
// global loads and stores of u, b and the traces are consecutive across
// lanes (dual form, see dual_sweep: x-lines).  In the nodal form, whose steps
// follow, the lifts of all facets are added where the state holds nodal
// values along every axis (b multiplied by Mhat^-1 along each axis), where a
// facet field needs no tangential transform (see nodal_lifts).  Steps of the
// fused sweep, one barrier after each (3D):
//   z  u, b lines and the neighbour traces -> registers; traces -> LDS;
//      Mhat^-1 b along z
//   y  Mhat^-1
//   x  Mhat^-1, minus the lifts of all facets, Si = S^T Mhat
//   z  Si
//   y  Si, division by the eigenvalue sums, S
//   x  S
//   z  S, update, store of u and of the z-facet traces
//   x, y facet traces from the updated cell in LDS
// The facet traces are written by each cell for its own interior facets and
// read once by the neighbour in the next sweep.  Where a block is a brick of
// cells (see brick), only the facets on its faces go through the buffers: two
// steps before the first one put u in LDS and hand the traces of the facets
// inside the brick from cell to cell.
#pragma once
#include <type_traits>

#include "dg_kernels.hpp"

// A translation unit compiles the cell kernels for one block shape (DGShapeV)
// by defining HPMG_TILE first: they live in namespace dgk (0) or
// dgk_t<HPMG_TILE>, and unqualified DGShape<D, N> names that shape.
#ifndef HPMG_TILE
#define HPMG_TILE 0
#endif
#if HPMG_TILE == 0
#define HPMG_DGK dgk
#else
#define HPMG_DGK_CAT2(a, b) a##b
#define HPMG_DGK_CAT(a, b) HPMG_DGK_CAT2(a, b)
#define HPMG_DGK HPMG_DGK_CAT(dgk_t, HPMG_TILE)
#endif

namespace hpmg {
namespace HPMG_DGK {
template <int D, int N>
using DGShape = ::hpmg::DGShapeV<D, N, HPMG_TILE>;

// Offset of the first node of the line of thread `ln` along axis k, and the
// node stride along that axis (x fastest).  The facet node index of the line
// on the facets normal to k is `ln` itself for every axis.
template <int D, int N>
__device__ __forceinline__ int line_base(int k, int ln) {
  if constexpr (D == 2) {
    return k == 0 ? N * ln : ln;
  } else {
    const int i0 = ln % N, i1 = ln / N;
    if (k == 0) return N * i0 + N * N * i1;
    if (k == 1) return i0 + N * N * i1;
    return i0 + N * i1;
  }
}
template <int N>
__device__ __forceinline__ constexpr int line_stride(int k) {
  return k == 0 ? 1 : (k == 1 ? N : N * N);
}

// The same for the cell data in LDS (padded rows, see DGShapeV::SY).
template <int D, int N>
__device__ __forceinline__ int lds_line(int cl, int k, int ln) {
  using Sh = DGShape<D, N>;
  if constexpr (D == 2) {
    return cl * Sh::NVP + (k == 0 ? Sh::SY * ln : ln);
  } else {
    const int i0 = ln % N, i1 = ln / N;
    return cl * Sh::NVP + (k == 0 ? Sh::SY * i0 + N * Sh::SY * i1 : (k == 1 ? i0 + N * Sh::SY * i1 : i0 + Sh::SY * i1));
  }
}
template <int D, int N>
__device__ __forceinline__ constexpr int lds_stride(int k) {
  return k == 0 ? 1 : (k == 1 ? DGShape<D, N>::SY : N * DGShape<D, N>::SY);
}

// Read-only data addressed uniformly across a wave: the constant address
// space lets the compiler fetch it with scalar loads into SGPRs.
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p) {
  // the same in every lane: without this the compiler keeps the pointer in
  // vector registers once some lanes have used it, and loads the tables per
  // lane (100 vector loads a wave in the FP64 degree-4 sweep)
  const unsigned long long v = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((int)v), hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
  return (cptr<T>)(((unsigned long long)hi << 32) | lo);
}

// out = G in, G row-major N x N (TR: G^T)
template <int N, bool TR, typename T, typename P>
__device__ __forceinline__ void mv(P G, const T (&in)[N], T (&out)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    T s = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) s += (TR ? G[j * N + i] : G[i * N + j]) * in[j];
    out[i] = s;
  }
}

// Even-odd products with matrices of mirror symmetry, from compact tables
// (EO<N>::SIZE entries, fetched with scalar loads): about half the
// multiply-adds and half the scalar registers of mv.
//
// S of the interior class holds mirror-even columns c < NE, then mirror-odd
// ones: table [i][c] = S(i, c) for i, c < NE, then [i][c] = S(i, NE + c) for
// i, c < H.  eo_fwd: out = S^T in (with the table of Si^T: out = Si in);
// eo_inv: out = S in.
template <int N>
struct EO {
  static constexpr int H = N / 2, NE = (N + 1) / 2, SIZE = NE * NE + H * H;
};
template <int N, typename T, typename P>
__device__ __forceinline__ void eo_fwd(P G, const T (&in)[N], T (&out)[N]) {
  constexpr int H = EO<N>::H, NE = EO<N>::NE;
  T e[H], o[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    e[i] = in[i] + in[N - 1 - i];
    o[i] = in[i] - in[N - 1 - i];
  }
#pragma unroll
  for (int c = 0; c < NE; ++c) {
    T s = (N & 1) ? G[H * NE + c] * in[H] : T(0);
#pragma unroll
    for (int i = 0; i < H; ++i) s += G[i * NE + c] * e[i];
    out[c] = s;
  }
#pragma unroll
  for (int c = 0; c < H; ++c) {
    T s = 0;
#pragma unroll
    for (int i = 0; i < H; ++i) s += G[NE * NE + i * H + c] * o[i];
    out[NE + c] = s;
  }
}
template <int N, typename T, typename P>
__device__ __forceinline__ void eo_inv(P G, const T (&in)[N], T (&out)[N]) {
  constexpr int H = EO<N>::H, NE = EO<N>::NE;
  T ev[NE], od[H];
#pragma unroll
  for (int i = 0; i < NE; ++i) {
    ev[i] = 0;
#pragma unroll
    for (int c = 0; c < NE; ++c) ev[i] += G[i * NE + c] * in[c];
  }
#pragma unroll
  for (int i = 0; i < H; ++i) {
    od[i] = 0;
#pragma unroll
    for (int c = 0; c < H; ++c) od[i] += G[NE * NE + i * H + c] * in[NE + c];
  }
  // out written in ascending order (as mv does), so that the stores of the
  // alternative paths of block_mv coincide index by index (no scratch)
#pragma unroll
  for (int i = 0; i < N; ++i)
    out[i] = i < H ? ev[i] + od[i] : (i == H && (N & 1) ? ev[H] : ev[N - 1 - i] - od[N - 1 - i]);
}
// x = G x for a matrix with G(N-1-i, N-1-j) = G(i, j) (Mhat and its inverse):
// table [i][j] = (G(i, j) + G(i, N-1-j)) / 2 for i, j < NE (G(i, H) in the
// middle column of odd N), then the halved differences for i, j < H.
template <int N, typename T, typename P>
__device__ __forceinline__ void cs_mv(P G, T (&x)[N]) {
  constexpr int H = EO<N>::H, NE = EO<N>::NE;
  T e[NE], o[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    e[i] = x[i] + x[N - 1 - i];
    o[i] = x[i] - x[N - 1 - i];
  }
  if (N & 1) e[NE - 1] = x[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    T ev = 0, od = 0;
#pragma unroll
    for (int j = 0; j < NE; ++j) ev += G[i * NE + j] * e[j];
#pragma unroll
    for (int j = 0; j < H; ++j) od += G[NE * NE + i * H + j] * o[j];
    x[i] = ev + od;
    x[N - 1 - i] = ev - od;
  }
  if (N & 1) {
    T ev = 0;
#pragma unroll
    for (int j = 0; j < NE; ++j) ev += G[H * NE + j] * e[j];
    x[H] = ev;
  }
}

template <int D>
__device__ __forceinline__ int ipow(int n, int k) {
  return k == 0 ? 1 : (k == 1 ? n : n * n);
}

// 1/d: hardware reciprocal refined by Newton steps (two for double, one for
// float) to full precision.
__device__ __forceinline__ double recip(double d) {
  double r = __builtin_amdgcn_rcp(d);
  r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
  r = __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
  return r;
}
__device__ __forceinline__ float recip(float d) {
  float r = __builtin_amdgcn_rcpf(d);
  return __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
}

// Thread index within the block's NT working threads; threads beyond NT
// (a batched launch uses one block size for every degree) get an index past
// every work range, so they only take part in the barriers.
template <int D, int N>
__device__ __forceinline__ int work_tid() {
  return threadIdx.x < DGShape<D, N>::NT ? (int)threadIdx.x : (1 << 28);
}

// Local cell and line of the thread (a cell index past the block's cells for
// a thread without a line).
template <int D, int N>
__device__ __forceinline__ void cell_line(int& cl, int& ln) {
  using Sh = DGShape<D, N>;
  if constexpr (Sh::WAVE) {
    const int lane = threadIdx.x & 63;
    cl = lane < Sh::CPW * Sh::L ? (int)(threadIdx.x >> 6) * Sh::CPW + lane / Sh::L : (1 << 20);
    ln = lane % Sh::L;
  } else {
    const int tid = work_tid<D, N>();
    cl = tid / Sh::L;
    ln = tid % Sh::L;
  }
}

// Barrier between two steps that exchange lines within each cell: of the
// block, or, where no cell is split between waves, of the wave, whose LDS
// accesses complete in program order (the fence keeps the compiler's).
template <int D, int N>
__device__ __forceinline__ void cell_sync() {
  if constexpr (DGShape<D, N>::WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// Boundary mask of a cell (bit f = 2k + side set: facet f on the domain
// boundary); the class of the cell along axis k is (mask >> 2k) & 3.
__device__ __forceinline__ int axis_class(int mask, int k) { return (mask >> (2 * k)) & 3; }

// Adaptive meshes (AD): the mask also holds bit 8 + f for a facet f that is
// the coarse side of a hanging facet (its penalty is r times the conforming
// one), and the class of axis k adds those two bits: 16 class tables.
template <bool AD>
__device__ __forceinline__ int axis_cls(int mask, int k) {
  if constexpr (AD)
    return ((mask >> (2 * k)) & 3) | (((mask >> (8 + 2 * k)) & 3) << 2);
  else
    return (mask >> (2 * k)) & 3;
}
template <bool AD>
constexpr int n_classes() {
  return AD ? 16 : 4;
}
template <bool AD, typename T>
__device__ __forceinline__ int cell_mask(const DGArgs<T>& a, int c) {
  if constexpr (AD)
    return a.amask[c];
  else
    return a.bmask[c];
}

// The cells of one block, by local index cl < CPB: a run of consecutive cells
// (2D, HPMG_TILE 3; id the block's number) or a brick (3D; id from brick_id),
// whose cells past the end of the mesh are not valid.
template <int D, int N, bool AD>
struct Cells {
  using Sh = DGShape<D, N>;
  static constexpr bool BR = D == 3 && HPMG_TILE != 3;
  static_assert(!BR || !AD, "adaptive meshes: runs of cells");
  int n, c0 = 0, nc = 0;                  // run: first cell, count
  int b[3], o[3], s[3];                   // brick: its place, first cell and cells per axis
  template <typename T>
  __device__ __forceinline__ Cells(const DGArgs<T>& a, int id) : n(a.n) {
    if constexpr (BR) {
      constexpr int B[3] = {Sh::BX, Sh::BY, Sh::BZ};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        b[k] = (id >> (10 * k)) & 1023;
        o[k] = b[k] * B[k];
        s[k] = min(B[k], n - o[k]);
      }
    } else {
      c0 = id * Sh::CPB;
      nc = min(Sh::CPB, a.ncell - c0);
    }
  }
  __device__ __forceinline__ void local(int cl, int (&l)[3]) const {
    l[0] = cl % Sh::BX;
    l[1] = cl / Sh::BX % Sh::BY;
    l[2] = cl / (Sh::BX * Sh::BY);
  }
  // local indices the block's loops run over (a brick's may be not valid)
  __device__ __forceinline__ int count() const { return BR ? Sh::CPB : nc; }
  __device__ __forceinline__ bool valid(int cl) const {
    if constexpr (BR) {
      int l[3];
      local(cl, l);
      return cl < Sh::CPB && l[0] < s[0] && l[1] < s[1] && l[2] < s[2];
    } else {
      return cl < nc;
    }
  }
  // its cell; for an index that is not valid another cell of the block
  __device__ __forceinline__ int cell(int cl) const {
    if constexpr (BR) {
      int l[3];
      local(min(cl, Sh::CPB - 1), l);
      return o[0] + min(l[0], s[0] - 1) + n * (o[1] + min(l[1], s[1] - 1) + n * (o[2] + min(l[2], s[2] - 1)));
    } else {
      return c0 + min(cl, nc - 1);
    }
  }
  // facet mask of cell c = cell(cl) (see axis_class, axis_cls)
  template <typename T>
  __device__ __forceinline__ int mask(const DGArgs<T>& a, int cl, int c) const {
    if constexpr (BR) {
      int l[3], m = 0;
      local(cl, l);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int x = o[k] + min(l[k], s[k] - 1);
        m |= (x == 0 ? 1 : 0) << (2 * k) | (x == n - 1 ? 1 : 0) << (2 * k + 1);
      }
      return m;
    } else {
      return cell_mask<AD>(a, c);
    }
  }
  // Brick: facet f of local cell l lies on the brick's face.
  __device__ __forceinline__ bool face(int f, const int (&l)[3]) const {
    const int k = f >> 1;
    return (f & 1) ? l[k] == s[k] - 1 : l[k] == 0;
  }
  // Brick: trace record of facet f on the brick's face, written by the cell
  // (own_rec) or by the neighbour across it (nb_rec).  Per axis the buffer
  // holds the layers of lower faces, then of upper faces, and in a layer the
  // facets of each brick's face one after another: a brick reads and writes
  // six contiguous runs.
  __device__ __forceinline__ unsigned face_rec(int k, int side, int layer, const int (&l)[3]) const {
    const int i = k == 0 ? 1 : 0, j = k == 2 ? 1 : 2;  // tangential axes
    const int nb[3] = {brick_layers(n, Sh::BX), brick_layers(n, Sh::BY), brick_layers(n, Sh::BZ)};
    const int before = k == 0 ? 0 : (k == 1 ? 2 * nb[0] : 2 * nb[0] + 2 * nb[1]);
    return (unsigned)(n * n) * (unsigned)(before + side * nb[k] + layer) +
           (unsigned)(o[j] * n + s[j] * o[i] + l[i] + s[i] * l[j]);
  }
  __device__ __forceinline__ unsigned own_rec(int f, const int (&l)[3]) const {
    return face_rec(f >> 1, f & 1, b[f >> 1], l);
  }
  __device__ __forceinline__ unsigned nb_rec(int f, const int (&l)[3]) const {
    return face_rec(f >> 1, (f & 1) ^ 1, b[f >> 1] + ((f & 1) ? 1 : -1), l);
  }
  // number of the block among the blocks of one right-hand side
  __device__ __forceinline__ int number(int id) const {
    if constexpr (BR)
      return b[0] + brick_layers(n, Sh::BX) * (b[1] + brick_layers(n, Sh::BY) * b[2]);
    else
      return id;
  }
};

// Block and right-hand side of a launch (block_grid).
template <int D, int N, bool AD, typename T>
__device__ __forceinline__ void block_of_grid(const DGArgs<T>& a, int& id, int& rhs) {
  if constexpr (Cells<D, N, AD>::BR) {
    const int nbx = brick_layers(a.n, DGShape<D, N>::BX);
    int x = blockIdx.x;
    rhs = 0;
    if (x >= nbx) {
      rhs = x / nbx;
      x -= rhs * nbx;
    }
    id = brick_id(x, blockIdx.y, blockIdx.z);
  } else {
    id = blockIdx.x;
    rhs = blockIdx.y;
  }
}

// LDS size of the staged eigendata: constant kappa shares the 4 (adaptive:
// 16) class tables, variable kappa stages S | lambda per cell and axis (2D:
// then the scratch of recompute_eig, which takes the trace slots in 3D).
template <int D, int N, bool VARK, bool AD = false>
struct EigLDS {
  static constexpr int SIZE =
      VARK ? DGShape<D, N>::CPB * D * (DGShape<D, N>::EGV + (D == 2 ? N * N : 0))
           : n_classes<AD>() * DGShape<D, N>::EGS;
};

// LDS after the staged eigendata: kappa_F per (cell, facet) (variable
// kappa; none otherwise), kappa_K per cell (variable kappa), the lift
// coefficients AL0 | BE0 (2N), then the boundary masks of the block's cells
// (matrix-core sweep).
template <int D, int N, bool VARK>
constexpr int kappa_lds_entries() {
  return (VARK ? DGShape<D, N>::CPB * (DGShape<D, N>::NF + 1) : 0) + 2 * N;
}
template <int D, int N, bool VARK, typename C>
__device__ __forceinline__ C* lift_lds(C* sKF) {
  return sKF + kappa_lds_entries<D, N, VARK>() - 2 * N;
}
template <int D, int N, bool VARK, typename C>
__device__ __forceinline__ int* mask_lds(C* sKF) {
  return (int*)(sKF + kappa_lds_entries<D, N, VARK>());
}
template <int D, int N, bool VARK, typename C>
__device__ __forceinline__ const int* mask_lds(const C* sKF) {
  return (const int*)(sKF + kappa_lds_entries<D, N, VARK>());
}

// Stage the eigendata (and, per cell, kappa_F of every facet; 0 on the
// boundary) of the block's cells.
template <typename T, int D, int N, bool VARK, bool AD = false, typename CellsT>
__device__ __forceinline__ void load_eig(const DGArgs<T>& a, const CellsT& B, CT<T>* sE, CT<T>* sKF) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int NN = N * N;
  const int tid = work_tid<D, N>();
  if constexpr (!VARK) {
    constexpr int NE = n_classes<AD>() * Sh::EGS, IE = (NE + Sh::NT - 1) / Sh::NT;
    C ev[IE];
#pragma unroll
    for (int m = 0; m < IE; ++m) ev[m] = a.eig[min(tid + m * Sh::NT, NE - 1)];
#pragma unroll
    for (int m = 0; m < IE; ++m)
      if (tid + m * Sh::NT < NE) sE[tid + m * Sh::NT] = ev[m];
  } else {
    // every load of the thread is issued before the first LDS store (no
    // load waits on another): eigendata, then kappa of the cell and of its
    // neighbour across each facet (the neighbour index is clamped into the
    // mesh so that it needs no boundary test; boundary facets get 0)
    constexpr int NE = Sh::CPB * D * (NN + N);
    constexpr int IE = (NE + Sh::NT - 1) / Sh::NT;
    constexpr int NK = Sh::CPB * Sh::NF;
    constexpr int IK = (NK + Sh::NT - 1) / Sh::NT;
    const int ne = B.count() * D * (NN + N), nk = B.count() * Sh::NF;
    C ev[IE], k0[IK], k1[IK];
    int msk[IK];
    const bool stored = a.rk == nullptr;  // else rebuilt by recompute_eig
#pragma unroll
    for (int m = 0; m < IE; ++m) {
      const int i = tid + m * Sh::NT;
      constexpr int R = D * (NN + N);  // words per cell
      ev[m] = (stored && i < ne) ? a.eig[(size_t)B.cell(i / R) * R + i % R] : C(0);
    }
#pragma unroll
    for (int m = 0; m < IK; ++m) {
      const int i = tid + m * Sh::NT;
      const int cl = i / Sh::NF, f = i % Sh::NF;
      const int c = B.cell(cl);
      const int st = ipow<D>(a.n, f >> 1);
      const int nb = min(max((f & 1) ? c + st : c - st, 0), a.ncell - 1);
      msk[m] = a.bmask[c];
      k0[m] = a.kappa[c];
      k1[m] = a.kappa[nb];
    }
#pragma unroll
    for (int m = 0; m < IE; ++m) {
      const int i = tid + m * Sh::NT;
      if (stored && i < ne) sE[i] = ev[m];
    }
#pragma unroll
    for (int m = 0; m < IK; ++m) {
      const int i = tid + m * Sh::NT;
      if (i < nk) {
        const int f = i % Sh::NF;
        sKF[i] = ((msk[m] >> f) & 1) ? C(0) : C(2) * k0[m] * k1[m] / (k0[m] + k1[m]);
        if (f == 0) sKF[Sh::CPB * Sh::NF + i / Sh::NF] = k0[m];  // kappa_K
      }
    }
  }
}

// Round-robin slot moves of the parallel Jacobi sweep: the slots 0 .. M - 2
// form a circle (position c sits in slot M - 2 for c = 0, in slot 2 (c - 1)
// for 1 <= c < M / 2, in slot 2 (M - 2 - c) + 1 otherwise), paired so that
// circle positions c and M - 1 - c share a slot pair and position 0 pairs
// with the fixed slot M - 1; one step moves position c to c + 1.
template <int M>
__host__ __device__ constexpr int jac_circle_slot(int c) {
  return c == 0 ? M - 2 : (c < M / 2 ? 2 * (c - 1) : 2 * (M - 2 - c) + 1);
}
template <int M>
__host__ __device__ constexpr int jac_slot_circle(int s) {
  return s == M - 2 ? 0 : ((s & 1) == 0 ? s / 2 + 1 : M - 2 - (s - 1) / 2);
}
template <int M>
__host__ __device__ constexpr int jac_next(int s) {
  return s == M - 1 ? s : jac_circle_slot<M>((jac_slot_circle<M>(s) + 1) % (M - 1));
}
template <int M>
__host__ __device__ constexpr int jac_prev(int s) {
  return s == M - 1 ? s : jac_circle_slot<M>((jac_slot_circle<M>(s) + M - 2) % (M - 1));
}

// Fast-diagonalisation data of every staged (cell, axis), rebuilt from kappa
// (block_recompute; the paper's variant that forms the block inverse anew in
// each cell and traversal), in the cell's own S | lambda record in LDS:
//   L   = kappa_K Khat + sum_s [c1_s (e_s ep_s^T + ep_s e_s^T) + c2_s e_s e_s^T]
//         (c1, c2) = (-kappa_F/2, sigma_hat kappa_F) interior, (-kappa_K,
//         2 sigma_hat kappa_K) on the boundary (a boundary facet has kappa_F 0)
//   A   = W L W^T with W = C^-1, Mhat = C C^T (symmetric), in scratch (N^2
//         words per cell and axis)
//   parallel Jacobi rotations A <- J^T A J, V <- V J (V in the S slot) until A
//   is diagonal to working precision (at most 8 sweeps in FP64, 6 in FP32)
//   lambda = diag(A), S = W^T V, so that L S = Mhat S diag(lambda), S^T Mhat S = I.
// N lanes of one wave share a (cell, axis): lane r owns row r of every
// product; the products that form A and S go through the cell's LDS record,
// and the rotations run in registers with cross-lane shuffles.  The lanes of
// a problem are in one wave, whose LDS accesses complete in program order,
// so a wavefront-scope fence between the phases orders them.
template <typename T, int D, int N>
__device__ __forceinline__ void recompute_eig(const DGArgs<T>& a, int nc, CT<T>* sE, const CT<T>* sKF,
                                              CT<T>* scratch) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int NN = N * N;
  constexpr int SWEEPS = sizeof(C) == 8 ? 8 : 6;
  // the block has NT threads (not always whole waves): its last wave hosts
  // only the problems whose N lanes all exist
  constexpr int TPW = 64 / N;  // problems per full wave
  constexpr int NWT = (Sh::NT + 63) / 64;
  constexpr int CLAST = (Sh::NT - 64 * (NWT - 1)) / N < TPW ? (Sh::NT - 64 * (NWT - 1)) / N : TPW;
  constexpr int CAP = (NWT - 1) * TPW + CLAST;  // problems per round of the block
  static_assert(CAP > 0, "no wave can host a problem");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane % N, slot = lane / N;
  const int cap_w = wave == NWT - 1 ? CLAST : TPW;
  const C* sKK = sKF + Sh::CPB * Sh::NF;
  const cptr<C> Kh = as_const(a.rk);
  const cptr<C> Wi = as_const(a.rk) + NN;
  const cptr<C> ev0 = as_const(a.ref) + RefOff<N>::EV0;
  const cptr<C> ev1 = as_const(a.ref) + RefOff<N>::EV1;
  const cptr<C> ep0 = as_const(a.ref) + RefOff<N>::EP0;
  const cptr<C> ep1 = as_const(a.ref) + RefOff<N>::EP1;
  const auto wave_sync = []() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); };
  // rounds of CAP problems; every lane of the block runs the same rounds
  for (int R = 0; R * CAP < nc * D; ++R) {
    const int t = R * CAP + wave * TPW + slot;
    const bool act = slot < cap_w && t < nc * D;
    if (__all(!act)) continue;  // nothing for this wave in this round
    const int tt = act ? t : R * CAP;  // idle lanes shadow a valid problem, writing nothing
    const int cl = tt / D, k = tt % D;
    C* V = sE + tt * Sh::EGV;
    C* A = scratch + tt * NN;
    C* lam = V + NN;
    const C kK = sKK[cl];
    const C kF0 = sKF[cl * Sh::NF + 2 * k], kF1 = sKF[cl * Sh::NF + 2 * k + 1];
    const bool b0 = kF0 == C(0), b1 = kF1 == C(0);
    const C c10 = b0 ? -kK : C(-0.5) * kF0, c20 = a.sigma_hat * (b0 ? C(2) * kK : kF0);
    const C c11 = b1 ? -kK : C(-0.5) * kF1, c21 = a.sigma_hat * (b1 ? C(2) * kK : kF1);
    // row r of L, of W L (into V), of A = (W L) W^T
    C row[N];
#pragma unroll
    for (int j = 0; j < N; ++j)
      row[j] = kK * Kh[r * N + j] + c10 * (ev0[r] * ep0[j] + ep0[r] * ev0[j]) + c20 * ev0[r] * ev0[j] +
               c11 * (ev1[r] * ep1[j] + ep1[r] * ev1[j]) + c21 * ev1[r] * ev1[j];
    if (act) {
#pragma unroll
      for (int j = 0; j < N; ++j) A[r * N + j] = row[j];
    }
    wave_sync();
#pragma unroll
    for (int j = 0; j < N; ++j) {
      C s = 0;
#pragma unroll
      for (int m = 0; m < N; ++m) s += Wi[r * N + m] * A[m * N + j];  // W lower triangular: zeros above
      row[j] = s;
    }
    wave_sync();
    if (act) {
#pragma unroll
      for (int j = 0; j < N; ++j) V[r * N + j] = row[j];
    }
    wave_sync();
#pragma unroll
    for (int j = 0; j < N; ++j) {
      C s = 0;
#pragma unroll
      for (int m = 0; m < N; ++m) s += V[r * N + m] * Wi[j * N + m];
      row[j] = s;
    }
    wave_sync();
    if (act) {
#pragma unroll
      for (int j = 0; j < N; ++j) A[r * N + j] = row[j];
#pragma unroll
      for (int j = 0; j < N; ++j) V[r * N + j] = j == r ? C(1) : C(0);
    }
    wave_sync();
    // symmetrise: A <- (A + A^T) / 2
#pragma unroll
    for (int j = 0; j < N; ++j) row[j] = C(0.5) * (A[r * N + j] + A[j * N + r]);
    wave_sync();
    if (act) {
#pragma unroll
      for (int j = 0; j < N; ++j) A[r * N + j] = row[j];
    }
    wave_sync();
    // Parallel Jacobi rotations in registers (round-robin ordering): the
    // rows and columns of A sit in M = N + (N & 1) slots; every round
    // rotates the disjoint slot pairs (2k, 2k+1) (for odd N slot N is an
    // empty placeholder, so slot N - 1 waits), then moves the indices one
    // step along a circle of the slots 0 .. M - 2 (slot M - 1 stays), so
    // that in M - 1 rounds every index pair meets once.  Lane r holds the
    // row of slot r of A and of V (V's rows stay in the original order, its
    // columns move with A's).  The order of the eigenpairs that results is
    // immaterial: lambda and the columns of S move together.
    constexpr int M = N + (N & 1);
    C arow[N], vrow[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      arow[j] = A[r * N + j];
      vrow[j] = j == r ? C(1) : C(0);
    }
    const int base = lane - r;  // lane of slot 0 of this problem
    const int pr = r ^ 1;       // partner slot
    const bool paired = pr < N;
    const bool lower = (r & 1) == 0;
    const int src_pair = base + (paired ? pr : r);
    const int src_move = base + jac_prev<M>(r);  // slot whose row moves into slot r
    bool done = !act;
#pragma unroll 1
    for (int sw = 0; sw < SWEEPS; ++sw) {
      // stop once the off-diagonal part is below working precision (every
      // lane of a problem forms the same sums)
      C offr = 0, dgr = 0;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        if (j == r)
          dgr = arow[j] * arow[j];
        else
          offr += arow[j] * arow[j];
      }
      C off = 0, dg = 0;
#pragma unroll
      for (int m = 0; m < N; ++m) {
        off += __shfl(offr, base + m, 64);
        dg += __shfl(dgr, base + m, 64);
      }
      done = done || C(0.5) * off <= (sizeof(C) == 8 ? C(1e-30) : C(1e-14)) * dg;
      if (__all(done)) break;  // every problem of the wave has converged
#pragma unroll 1
      for (int t = 0; t < M - 1; ++t) {
        C mydiag = 0, myoff = 0;
#pragma unroll
        for (int j = 0; j < N; ++j) {
          if (j == r) mydiag = arow[j];
          if (j == pr) myoff = arow[j];
        }
        const C pdiag = __shfl(mydiag, src_pair, 64);
        const C poff = __shfl(myoff, src_pair, 64);
        // both lanes of a pair form the angle from the lower slot's entry
        const C app = lower ? mydiag : pdiag, aqq = lower ? pdiag : mydiag, apq = lower ? myoff : poff;
        // an unpaired, converged or already zero pair rotates by the identity
        const bool rot = paired && !done && apq != C(0);
        const C tau = (aqq - app) / (C(2) * (rot ? apq : C(1)));
        const C at = __builtin_fabs(tau);
        // t = sign(tau) / (|tau| + sqrt(1 + tau^2)), without overflow
        const C ia = C(1) / (at > C(1) ? at : C(1));
        const C root = at > C(1) ? at * __builtin_sqrt(C(1) + ia * ia) : __builtin_sqrt(C(1) + at * at);
        const C tn = __builtin_copysign(C(1), tau) / (at + root);
        const C cs = rot ? C(1) / __builtin_sqrt(C(1) + tn * tn) : C(1);
        const C sn = rot ? tn * cs : C(0);
        // columns 2k, 2k+1 of the rows of A and V (the pair's angle is held
        // by the lane of slot 2k)
#pragma unroll
        for (int k = 0; 2 * k + 1 < N; ++k) {
          const C cj = __shfl(cs, base + 2 * k, 64), sj = __shfl(sn, base + 2 * k, 64);
          const C x = arow[2 * k], y = arow[2 * k + 1];
          arow[2 * k] = cj * x - sj * y;
          arow[2 * k + 1] = sj * x + cj * y;
          const C vx = vrow[2 * k], vy = vrow[2 * k + 1];
          vrow[2 * k] = cj * vx - sj * vy;
          vrow[2 * k + 1] = sj * vx + cj * vy;
        }
        // rows: p' = cs p - sn q, q' = sn p + cs q; the pair's entry is zero
        // afterwards
        const C so = lower ? -sn : sn;  // coefficient of the partner's row
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const C pj = __shfl(arow[j], src_pair, 64);
          const C nv = cs * arow[j] + so * pj;
          arow[j] = (rot && j == pr) ? C(0) : nv;
        }
        // move every index one step along the circle: row of slot prev(r)
        // into slot r, column j into column next(j)
        C na[N], nvr[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
          na[jac_next<M>(j)] = __shfl(arow[j], src_move, 64);
          nvr[jac_next<M>(j)] = vrow[j];
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
          arow[j] = na[j];
          vrow[j] = nvr[j];
        }
      }
    }
    wave_sync();
    if (act) {
#pragma unroll
      for (int j = 0; j < N; ++j) {
        A[r * N + j] = arow[j];
        V[r * N + j] = vrow[j];
      }
    }
    wave_sync();
    // lambda = diag(A); S = W^T V, row r: S[r][c] = sum_{m >= r} W[m][r] V[m][c]
    const C lr = A[r * N + r];
#pragma unroll
    for (int c = 0; c < N; ++c) {
      C s = 0;
#pragma unroll
      for (int m = 0; m < N; ++m) s += Wi[m * N + r] * V[m * N + c];
      row[c] = s;
    }
    wave_sync();
    if (act) {
      lam[r] = lr;
#pragma unroll
      for (int c = 0; c < N; ++c) V[r * N + c] = row[c];
    }
    wave_sync();
  }
}

// Variable kappa, apply (EV): S of every staged record becomes Si = S^T Mhat,
// each entry rounded once as in the class tables (as two products an apply to
// a smooth u has up to 1.25 times the error).  Follows a barrier that has
// staged the records; one more must follow.
template <typename T, int D, int N>
__device__ __forceinline__ void make_si(const DGArgs<T>& a, int nc, CT<T>* sE) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int R = (Sh::CPB * D * N + Sh::NT - 1) / Sh::NT;
  const cptr<C> Mh = as_const(a.ref) + RefOff<N>::M;
  const int tid = work_tid<D, N>();
  C x[R][N];  // row i % N of Si from that column of S
#pragma unroll
  for (int m = 0; m < R; ++m) {
    const int i = tid + m * Sh::NT;
    if (i >= nc * D * N) continue;
    const C* S = sE + i / N * Sh::EGV + i % N;
    C y[N];
#pragma unroll
    for (int j = 0; j < N; ++j) y[j] = S[j * N];
    mv<N, true>(Mh, y, x[m]);
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < R; ++m) {
    const int i = tid + m * Sh::NT;
    if (i >= nc * D * N) continue;
    C* E = sE + i / N * Sh::EGV + i % N * N;
#pragma unroll
    for (int j = 0; j < N; ++j) E[j] = x[m][j];
  }
}

// Matrix of (cell, axis k) applied to a line: S^T (OP_ST), Si = S^T Mhat
// (OP_SI), Si^T (OP_SIT) or S (OP_S).  Constant kappa: when every lane of the
// wave needs the interior class, the even-odd form from the compact tables;
// otherwise the class record's LDS copy.  Variable kappa: the cell's record,
// which holds S (then Si is two products, the first with Mhat) or, EV, Si.
enum BlockOp { OP_ST = 0, OP_SI = 1, OP_S = 2, OP_SIT = 3 };
template <typename T, int D, int N, bool VARK, bool IVAR, bool AD, int OP, bool EV = false>
__device__ __forceinline__ void block_mv(const DGArgs<T>& a, const CT<T>* sE, int cl, int mask, int k,
                                         const CT<T> (&in)[N], CT<T> (&out)[N]) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr bool si = OP == OP_SI || OP == OP_SIT, tr = OP == OP_ST || OP == OP_SIT;
  constexpr int off = si ? N * N : 0;
  if constexpr (VARK) {
    const C* G = sE + (cl * D + k) * Sh::EGV;
    static_assert(EV ? si : OP != OP_SIT, "matrix of the record");
    if constexpr (OP == OP_SI && !EV) {
      C x[N];
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = in[j];
      cs_mv<N>(as_const(a.ref) + RefOff<N>::MC, x);
      mv<N, true>(G, x, out);
    } else {
      mv<N, tr>(G, in, out);
    }
  } else {
    const int cls = IVAR ? 0 : axis_cls<AD>(mask, k);
    // 2D: FP32 of degree 8 is faster with the plain product on all but large
    // meshes (sweeps, even-odd against plain: 1.14 on 4^2 cells, 1.04 on 64^2,
    // 0.87 on 150^2; the errors are alike), FP64 of degree 6 to 8 on meshes of few blocks
    // (HPMG_TILE 4, see dg_inst_2d_double_plain.hip)
    // 3D runs of cells (HPMG_TILE 3: small and adaptive meshes) in FP64 and FP32: the
    // same trade at degree 6 to 8 and 8 (even-odd | plain, FP64 degree 6, 6^3 48 | 41
    // us, degree 7, 4^3 45 | 40, FP32 degree 8, 6^3 47 | 41)
    constexpr bool big = N > (sizeof(C) == 8 ? 6 : 8);
    constexpr bool eo = !big || (D == 3 ? HPMG_TILE != 3 || sizeof(T) == 2 : sizeof(C) == 8 && HPMG_TILE != 4);
    if (eo && (IVAR || __all(cls == 0))) {
      const cptr<C> G = as_const(a.ref) + (si ? RefOff<N>::SIC : RefOff<N>::SC);
      if constexpr (OP == OP_S || OP == OP_SIT)
        eo_inv<N>(G, in, out);
      else
        eo_fwd<N>(G, in, out);
    } else {
      mv<N, tr>(sE + cls * Sh::EGS + off, in, out);
    }
  }
}

// Eigenvalue sums of the line along axis k of thread line ln: out[j] =
// lambda_k[j] + the two (one) tangential eigenvalues.
template <int D, int N, bool VARK, bool IVAR, bool AD, typename C>
__device__ __forceinline__ void eig_sums(const C* sE, int cl, int mask, int k, int ln, C (&out)[N]) {
  using Sh = DGShape<D, N>;
  constexpr int NN = N * N;
  auto lam = [&](int m) -> const C* {
    return VARK ? sE + (cl * D + m) * Sh::EGV + NN : sE + (IVAR ? 0 : axis_cls<AD>(mask, m)) * Sh::EGS + 2 * NN;
  };
  C ls;
  if constexpr (D == 2)
    ls = lam(1 - k)[ln];
  else
    ls = lam(k == 0 ? 1 : 0)[ln % N] + lam(k == 2 ? 1 : 2)[ln / N];
  const C* lk = lam(k);
#pragma unroll
  for (int j = 0; j < N; ++j) out[j] = ls + lk[j];
}

// Trace record of a (facet, cell): L pairs (value g, reference outward
// normal derivative q), one per facet node.
template <typename T>
struct alignas(2 * sizeof(T)) TrPair {
  T g, q;
};

// Trace record (unit 2L values) that holds the neighbour-side traces of facet f
// of cell c in runs of cells.  A boundary facet has none (finish_pair zeroes
// what this names).  AD (adaptive meshes): the slot table names the record.
// IVAR (interior-block smoother): a boundary facet takes the cell's own traces,
// negated.
template <typename T, int D, int N, bool IVAR, bool AD>
__device__ __forceinline__ size_t nb_slot(const DGArgs<T>& a, int c, int mask, int f) {
  if constexpr (AD) {
    return (size_t)a.nbslot[(size_t)f * a.ncell + c];
  } else {
    const int st = ipow<D>(a.n, f >> 1);
    const int nb = min(max((f & 1) ? c + st : c - st, 0), a.ncell - 1);
    return IVAR && ((mask >> f) & 1) ? (size_t)f * a.ncell + c : (size_t)(f ^ 1) * a.ncell + nb;
  }
}
// The traces of cell c at facet node ln of every facet.
template <typename T, int D, int N, bool IVAR, bool AD>
__device__ __forceinline__ void load_pairs(const DGArgs<T>& a, const T* tr, int c, int mask, int ln,
                                           TrPair<T> (&p)[2 * D]) {
  constexpr int L = DGShape<D, N>::L;
#pragma unroll
  for (int f = 0; f < 2 * D; ++f)
    p[f] = *reinterpret_cast<const TrPair<T>*>(tr + (nb_slot<T, D, N, IVAR, AD>(a, c, mask, f) * L + ln) * 2);
}
// The pair as the lifts read it: zero (IVAR: negated) on a boundary facet;
// on the coarse side of a hanging facet, whose penalty is sig_hang,
// alpha q + beta g with the conforming coefficients needs
// q - 2 (sig_hang - sigma_hat) g.
template <typename T, bool IVAR, bool AD>
__device__ __forceinline__ TrPair<CT<T>> finish_pair(const DGArgs<T>& a, const TrPair<T>& p, int mask, int f) {
  using C = CT<T>;
  const bool bdy = (mask >> f) & 1;
  TrPair<C> r;
  r.g = (C)p.g;
  r.q = (C)p.q;
  if (bdy) {
    r.g = IVAR ? -r.g : C(0);
    r.q = IVAR ? -r.q : C(0);
  }
  if constexpr (AD) {
    if ((mask >> (8 + f)) & 1) r.q -= C(2) * (a.sig_hang - a.sigma_hat) * r.g;
  }
  return r;
}

// r += SIGN x the lifts of all facets at the nodes of the line along axis k
// of thread line ln, in nodal values (the dual lift of facet (m, s) is the
// facet mass times kappa_F (q'/2 - sigma_hat g') e_s + kappa_F g'/2 ep_s along
// its axis; multiplied by Mhat^-1 along every axis the mass cancels and the
// lift at a node is alpha_s q' + beta_s g' of the facet node it projects to,
//   alpha_s = kappa_F/2 Mhat^-1 e_s,
//   beta_s = kappa_F (Mhat^-1 ep_s / 2 - sigma_hat Mhat^-1 e_s),
// tables AL0, BE0 for s = 0 (kappa_F = 1 when it varies), mirrored for s = 1.
template <typename T, int D, int N, bool VARK, int SIGN>
__device__ __forceinline__ void nodal_lifts(const DGArgs<T>& a, int cl, int k, int ln, const CT<T>* sNB,
                                            const CT<T>* sKF, CT<T> (&r)[N]) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  constexpr C sg = C(SIGN);
  using P = TrPair<C>;
  const P* nb = reinterpret_cast<const P*>(sNB) + cl * Sh::NF * L;
  const C* kf = sKF + cl * Sh::NF;  // VARK only
  {
    const cptr<C> al = as_const(a.ref) + RefOff<N>::AL0;
    const cptr<C> be = as_const(a.ref) + RefOff<N>::BE0;
    P p0 = nb[(2 * k) * L + ln], p1 = nb[(2 * k + 1) * L + ln];
    const C f0 = VARK ? sg * kf[2 * k] : sg, f1 = VARK ? sg * kf[2 * k + 1] : sg;
    p0.g *= f0;
    p0.q *= f0;
    p1.g *= f1;
    p1.q *= f1;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      r[j] += al[j] * p0.q + be[j] * p0.g;
      r[j] += al[N - 1 - j] * p1.q + be[N - 1 - j] * p1.g;
    }
  }
  const C* sAB = sKF + kappa_lds_entries<D, N, VARK>() - 2 * N;
  static_assert(D == 3, "nodal form: 3D");
  const int i0 = ln % N, i1 = ln / N;
#pragma unroll
  for (int mm = 1; mm < D; ++mm) {
    // m: the other axes in increasing order; x = the line's index along m,
    // y = its index along the remaining axis
    const int m = mm - 1 < k ? mm - 1 : mm;
    const int x = mm == 1 ? i0 : i1, y = mm == 1 ? i1 : i0;
    // facet nodes of the line on the facets normal to m: the tangential axes
    // are k and the remaining one, lower axis first
    const int rest = 3 - k - m;
    const int base = k < rest ? N * y : y, st = k < rest ? 1 : N;
    const C f0 = VARK ? sg * kf[2 * m] : sg, f1 = VARK ? sg * kf[2 * m + 1] : sg;
    const C a0 = f0 * sAB[x], b0 = f0 * sAB[N + x], a1 = f1 * sAB[N - 1 - x], b1 = f1 * sAB[2 * N - 1 - x];
    const P* q0 = nb + (2 * m) * L + base;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const P p0 = q0[j * st], p1 = q0[L + j * st];
      r[j] += a0 * p0.q + b0 * p0.g;
      r[j] += a1 * p1.q + b1 * p1.g;
    }
  }
}

// Traces (value g, outward normal derivative d) of a line at its two ends.
template <typename T, int N>
__device__ __forceinline__ void line_traces(const DGArgs<T>& a, const CT<T> (&u)[N], CT<T>& g0, CT<T>& d0, CT<T>& g1,
                                            CT<T>& d1) {
  using C = CT<T>;
  const cptr<C> ep0 = as_const(a.ref) + RefOff<N>::EP0;
  const cptr<C> ep1 = as_const(a.ref) + RefOff<N>::EP1;
  d0 = 0;
  d1 = 0;
  g0 = u[0];
  g1 = u[N - 1];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    d0 += ep0[j] * u[j];
    d1 += ep1[j] * u[j];
  }
  if (a.gl) {  // value functionals are dense (Gauss-Legendre nodes)
    const cptr<C> ev0 = as_const(a.ref) + RefOff<N>::EV0;
    const cptr<C> ev1 = as_const(a.ref) + RefOff<N>::EV1;
    g0 = 0;
    g1 = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      g0 += ev0[j] * u[j];
      g1 += ev1[j] * u[j];
    }
  }
}

// The traces of a line along axis k, stored straight to the trace buffer
// where a neighbour reads them there: on the facets that are not on the
// boundary (bricks: on the faces of the brick).
template <typename T, int D, int N, bool IVAR, bool AD>
__device__ __forceinline__ void store_line_traces(const DGArgs<T>& a, T* trout, const Cells<D, N, AD>& B, int cl, int c,
                                                  int mask, int k, int ln, const CT<T> (&u)[N]) {
  using C = CT<T>;
  constexpr int L = DGShape<D, N>::L;
  C g0, d0, g1, d1;
  line_traces<T, N>(a, u, g0, d0, g1, d1);
  if constexpr (Cells<D, N, AD>::BR) {
    int l[3];
    B.local(cl, l);
    if (B.face(2 * k, l) && !((mask >> (2 * k)) & 1))
      *reinterpret_cast<TrPair<T>*>(trout + ((size_t)B.own_rec(2 * k, l) * L + ln) * 2) = {(T)g0, (T)d0};
    if (B.face(2 * k + 1, l) && !((mask >> (2 * k + 1)) & 1))
      *reinterpret_cast<TrPair<T>*>(trout + ((size_t)B.own_rec(2 * k + 1, l) * L + ln) * 2) = {(T)g1, (T)d1};
  } else {
    if (IVAR || !((mask >> (2 * k)) & 1))
      *reinterpret_cast<TrPair<T>*>(trout + (((size_t)(2 * k) * a.ncell + c) * L + ln) * 2) = {(T)g0, (T)d0};
    if (IVAR || !((mask >> (2 * k + 1)) & 1))
      *reinterpret_cast<TrPair<T>*>(trout + (((size_t)(2 * k + 1) * a.ncell + c) * L + ln) * 2) = {(T)g1, (T)d1};
  }
}

// Traces along every axis but F of the cell vector staged in sU.
template <typename T, int D, int N, int F, bool IVAR, bool AD>
__device__ __forceinline__ void store_other_traces(const DGArgs<T>& a, T* trout, const CT<T>* sU,
                                                   const Cells<D, N, AD>& B, int cl, int c, int mask, int ln) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    if (k == F) continue;
    const int base = lds_line<D, N>(cl, k, ln);
    C u[N];
#pragma unroll
    for (int j = 0; j < N; ++j) u[j] = sU[base + j * lds_stride<D, N>(k)];
    store_line_traces<T, D, N, IVAR>(a, trout, B, cl, c, mask, k, ln, u);
  }
}

// ---- dual form: facet transforms (also of the matrix-core sweep)

// Tangential axis of pass `pass` of the facet transform of facets normal to k.
template <int D>
__device__ __forceinline__ int tangential(int k, int pass) {
  if constexpr (D == 2)
    return 1 - k;
  else
    return pass == 0 ? ((k == 0) ? 1 : 0) : ((k == 2) ? 1 : 2);
}

// Facet flux fields.  From the neighbour's traces (g', q') across facet f
//   F1 = T_f (kappa_F (q'/2 - sigma_hat g')),  F2 = T_f (kappa_F g'/2),
// T_f = G_t1 x G_t2 over the tangential axes with G_t = Si_t for t < k
// (axes already transformed when facet k is processed) and Mhat otherwise.
// sNB[cl][f][F1|F2][L].  Pass 0 takes the traces [as g | q] and transforms along
// t1; pass 1 transforms along t2 (3D).  Work items are ordered (facet, cell,
// line) so that a wave mostly sees one facet direction and therefore one
// matrix.
//
// A line of facet f of local cell cl: pass 0's fluxes, then the matrix along t.
template <typename T, int D, int N, bool VARK, bool IVAR, bool AD, bool EV>
__device__ __forceinline__ void facet_line(const DGArgs<T>& a, int pass, const CT<T>* sE, const CT<T>* sKF, int cl,
                                           int f, int smask, CT<T> (&x1)[N], CT<T> (&x2)[N], CT<T> (&o1)[N],
                                           CT<T> (&o2)[N]) {
  using C = CT<T>;
  const int k = f >> 1, t = tangential<D>(k, pass);
  if (pass == 0) {
    const C kf = VARK ? sKF[cl * DGShape<D, N>::NF + f] : a.kappa_const;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const C gv = x1[j], qv = x2[j];
      // one rounding: sigma_hat g' and q'/2 cancel for a smooth u
      x1[j] = kf * fma(-a.sigma_hat, gv, C(0.5) * qv);
      x2[j] = C(0.5) * kf * gv;
    }
  }
  if (t < k) {
    block_mv<T, D, N, VARK, IVAR, AD, OP_SI, EV>(a, sE, cl, smask, t, x1, o1);
    block_mv<T, D, N, VARK, IVAR, AD, OP_SI, EV>(a, sE, cl, smask, t, x2, o2);
  } else {
    const cptr<C> Mh = as_const(a.ref) + RefOff<N>::M;
    mv<N, false>(Mh, x1, o1);
    mv<N, false>(Mh, x2, o2);
  }
}
template <typename T, int D, int N, bool VARK, bool IVAR, bool AD = false, bool EV = false>
__device__ __forceinline__ void facet_pass(const DGArgs<T>& a, const Cells<D, N, AD>& B, int pass, CT<T>* sNB,
                                           const CT<T>* sE, const CT<T>* sKF) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  constexpr int LINES = (D == 2) ? 1 : N;
  for (int i = work_tid<D, N>(); i < Sh::CPB * Sh::NF * LINES; i += Sh::NT) {
    const int f = i / (Sh::CPB * LINES), rem = i % (Sh::CPB * LINES);
    const int cl = rem / LINES, li = rem % LINES;
    if (!B.valid(cl)) continue;
    const int st = pass == 0 ? 1 : N;  // node stride along t within the facet
    C* g = sNB + (cl * Sh::NF + f) * 2 * L + (pass == 0 ? N * li : li);
    const int smask = IVAR ? 0 : mask_lds<D, N, VARK>(sKF)[cl];  // boundary classes of the block solve
    C x1[N], x2[N], o1[N], o2[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      x1[j] = g[st * j];
      x2[j] = g[L + st * j];
    }
    facet_line<T, D, N, VARK, IVAR, AD, EV>(a, pass, sE, sKF, cl, f, smask, x1, x2, o1, o2);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      g[st * j] = o1[j];
      g[L + st * j] = o2[j];
    }
  }
}

// Runs of cells with constant kappa take pass 0 straight from the trace buffer
// (FacetLoad): a barrier and an LDS round trip less than through staged traces
// (four matrix-core sweeps, FP16, Q4 32^3 237 -> 180 us, Q8 8^3 126 -> 83 us).  With variable kappa the pass needs the staged records.
template <int D, int N, bool VARK, bool AD>
constexpr bool pass0_on_load() {
  return !VARK && !Cells<D, N, AD>::BR;
}
// A thread's items of pass 0: every load is issued by the constructor, run()
// transforms them into sNB.
template <typename T, int D, int N, bool IVAR, bool AD>
struct FacetLoad {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  static constexpr int L = Sh::L, LINES = (D == 2) ? 1 : N, ITEMS = Sh::CPB * Sh::NF * LINES;
  static constexpr int IT = (ITEMS + Sh::NT - 1) / Sh::NT;
  TrPair<T> p[IT][N];
  int msk[IT];
  static __device__ __forceinline__ void item(const Cells<D, N, AD>& B, int m, int& f, int& cl, int& li, bool& ok) {
    const int i = work_tid<D, N>() + m * Sh::NT;
    f = min(i / (Sh::CPB * LINES), Sh::NF - 1);
    cl = i % (Sh::CPB * LINES) / LINES;
    li = i % LINES;
    ok = i < ITEMS && B.valid(cl);
  }
  __device__ __forceinline__ FacetLoad(const DGArgs<T>& a, const T* tr, const Cells<D, N, AD>& B) {
#pragma unroll
    for (int m = 0; m < IT; ++m) {
      int f, cl, li;
      bool ok;
      item(B, m, f, cl, li, ok);
      const int c = B.cell(ok ? cl : 0);
      msk[m] = cell_mask<AD>(a, c);
      const TrPair<T>* src =
          reinterpret_cast<const TrPair<T>*>(tr) + nb_slot<T, D, N, IVAR, AD>(a, c, msk[m], f) * L + N * li;
#pragma unroll
      for (int j = 0; j < N; ++j) p[m][j] = src[j];
    }
  }
  __device__ __forceinline__ void run(const DGArgs<T>& a, const Cells<D, N, AD>& B, C* sNB) const {
#pragma unroll
    for (int m = 0; m < IT; ++m) {
      int f, cl, li;
      bool ok;
      item(B, m, f, cl, li, ok);
      if (!ok) continue;
      C x1[N], x2[N], o1[N], o2[N];
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const TrPair<C> v = finish_pair<T, IVAR, AD>(a, p[m][j], msk[m], f);
        x1[j] = v.g;
        x2[j] = v.q;
      }
      // the class tables in global memory: those in LDS are not staged yet
      facet_line<T, D, N, false, IVAR, AD, false>(a, 0, a.eig, nullptr, cl, f, IVAR ? 0 : msk[m], x1, x2, o1, o2);
      C* g = sNB + (cl * Sh::NF + f) * 2 * L + N * li;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        g[j] = o1[j];
        g[L + j] = o2[j];
      }
    }
  }
};

// Staged trace of (local cell, facet) at facet node ln; SPLIT (dual form): the
// record as [g | q] instead of pairs.
template <int D, int N, bool SPLIT, typename C>
__device__ __forceinline__ void put_pair(C* sNB, int cl, int f, int ln, const TrPair<C>& v) {
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  if constexpr (SPLIT) {
    C* g = sNB + (cl * Sh::NF + f) * 2 * L + ln;
    g[0] = v.g;
    g[L] = v.q;
  } else {
    reinterpret_cast<TrPair<C>*>(sNB)[(cl * Sh::NF + f) * L + ln] = v;
  }
}

// Stages what a traversal of one block needs in LDS: the neighbour traces,
// the eigendata and the lift coefficients (a barrier must follow before they
// are read or sW is written).  The loads of a thread are all issued before
// the first LDS store.  Bricks: the traces at the brick's faces come from the
// buffer, those inside it from the block's own u (u: the thread's line along
// axis F), in storage precision as if they had been stored; sW is used.  EV:
// variable kappa's records as the apply reads them.  Where pass0_on_load, sNB
// gets the fields after pass 0 of the dual form's transforms instead.
template <typename T, int D, int N, bool VARK, bool IVAR, bool AD, bool TRACES, bool SPLIT, int F, bool EV = false>
__device__ __forceinline__ void stage_block(const DGArgs<T>& a, const T* tr, const Cells<D, N, AD>& B, int cl, int c,
                                            int ln, bool act, int mask, const CT<T> (&u)[N], CT<T>* sNB, CT<T>* sW,
                                            CT<T>* sE, CT<T>* sKF) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  constexpr bool BR = Cells<D, N, AD>::BR;
  const int tid = work_tid<D, N>();
  if constexpr (TRACES && SPLIT && pass0_on_load<D, N, VARK, AD>()) {
    const FacetLoad<T, D, N, IVAR, AD> fl(a, tr, B);
    load_eig<T, D, N, VARK, AD>(a, B, sE, sKF);
    fl.run(a, B, sNB);
    return;
  }
  TrPair<T> p[2 * D];
  int l[3] = {0, 0, 0};
  if constexpr (BR && TRACES) {
    B.local(act ? cl : 0, l);
#pragma unroll
    for (int f = 0; f < 2 * D; ++f) {
      p[f] = {T(0), T(0)};
      if (act && B.face(f, l) && !((mask >> f) & 1))
        p[f] = *reinterpret_cast<const TrPair<T>*>(tr + ((size_t)B.nb_rec(f, l) * L + ln) * 2);
    }
  } else if constexpr (TRACES) {
    load_pairs<T, D, N, IVAR, AD>(a, tr, c, mask, ln, p);
  }
  C* sAB = lift_lds<D, N, VARK>(sKF);
  const C ab = tid < 2 * N ? a.ref[RefOff<N>::AL0 + tid] : C(0);
  static_assert(2 * N <= Sh::NT, "the lift table is staged in one pass");
  load_eig<T, D, N, VARK, AD>(a, B, sE, sKF);
  if (tid < 2 * N) sAB[tid] = ab;
  if constexpr (VARK) {
    if (a.rk) {
      __syncthreads();
      recompute_eig<T, D, N>(a, B.count(), sE, sKF, D == 2 ? sE + Sh::CPB * D * Sh::EGV : sNB);
      __syncthreads();
    }
  }
  if constexpr (BR && TRACES) {
    if (act) {
      const int base = lds_line<D, N>(cl, F, ln);
#pragma unroll
      for (int j = 0; j < N; ++j) sW[base + j * lds_stride<D, N>(F)] = u[j];
#pragma unroll
      for (int f = 0; f < 2 * D; ++f)
        if (B.face(f, l) && !(IVAR && ((mask >> f) & 1)))
          put_pair<D, N, SPLIT>(sNB, cl, f, ln, TrPair<C>{(C)p[f].g, (C)p[f].q});
    }
  } else if constexpr (TRACES) {
    if (act) {
#pragma unroll
      for (int f = 0; f < 2 * D; ++f) put_pair<D, N, SPLIT>(sNB, cl, f, ln, finish_pair<T, IVAR, AD>(a, p[f], mask, f));
    }
  }
  if constexpr (BR && TRACES) {
    __syncthreads();
    if (act) {
#pragma unroll
      for (int k = 0; k < D; ++k) {
        C x[N];
        const int base = lds_line<D, N>(cl, k, ln);
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] = k == F ? u[j] : sW[base + j * lds_stride<D, N>(k)];
        constexpr int step[3] = {1, Sh::BX, Sh::BX * Sh::BY};
        C g0, d0, g1, d1;
        line_traces<T, N>(a, x, g0, d0, g1, d1);
        // rounded to the storage type, as a stored trace is
        const TrPair<C> q0 = {(C)(T)g0, (C)(T)d0}, q1 = {(C)(T)g1, (C)(T)d1};
        // the lower facet's trace is read by the cell below, and vice versa;
        // the interior-block smoother reads the cell's own, negated, at the
        // boundary
        if (!B.face(2 * k, l))
          put_pair<D, N, SPLIT>(sNB, cl - step[k], 2 * k + 1, ln, q0);
        else if (IVAR && ((mask >> (2 * k)) & 1))
          put_pair<D, N, SPLIT>(sNB, cl, 2 * k, ln, TrPair<C>{-q0.g, -q0.q});
        if (!B.face(2 * k + 1, l))
          put_pair<D, N, SPLIT>(sNB, cl + step[k], 2 * k, ln, q1);
        else if (IVAR && ((mask >> (2 * k + 1)) & 1))
          put_pair<D, N, SPLIT>(sNB, cl, 2 * k + 1, ln, TrPair<C>{-q1.g, -q1.q});
      }
    }
  }
  if constexpr (VARK && EV) {
    if constexpr (!(BR && TRACES)) __syncthreads();  // records staged
    make_si<T, D, N>(a, B.count(), sE);
  }
}

// Form of a traversal: nodal (sweep_body, apply_body) or dual
// (sweep_dual_body, apply_dual_body).  The nodal form is the faster one in 3D
// (see below), but the products with Mhat^-1 and Mhat add rounding, and with
// the tables rounded once for all cells the error is systematic: its ratio to
// the dual form's hardly depends on the mesh.  So a traversal is nodal where
// its error against 64 bits is no larger than the dual form's (within 5%, as
// far as the means below repeat).  Ratio at degree 1 to 8, four sweeps or one
// apply on 4^3 to 32^3 cells, constant kappa, for a random | a smooth u:
//   sweep FP64   .77  .96 1.04 1.01  .96 1.04 1.04 1.07 |  .58  .94 1.03 1.05  .96 1.77 1.21 2.01
//   sweep FP32  1.40 1.03 1.26 1.04  .78  .96 1.17 1.01 | 1.02  .57 1.15  .94  .92 1.96 2.64 1.35
//   apply FP64  1.11  .93 1.13  .98 1.00 1.02 1.02 1.02 | 2.39 1.03 1.23  .82  .93  .94  .74  .94
//   apply FP32  1.33 1.71 1.38 1.55 1.20 1.10 1.34 1.31 |  .81  .84  .98 1.19  .80 1.13  .98 1.01
// Variable kappa: sweeps .9 to 1.08 in FP64, 1.3 to 1.7 in FP32 at every degree;
// apply 1.2 and more at half of the degrees.  16-bit storage, whose stored u is
// coarser than either: 1.00 for sweeps; its residual, which steers the outer
// iteration, is dual (Q5 96^3, log-normal kappa, to 1e-9, with the outer
// residual in the same form: 40 iterations in FP16, 49 in BF16; nodal 42, and
// 56 without getting there).  Gauss-Legendre nodes (DGArgs::gl; FP64 and FP32)
// are dual throughout, by kernels of their own (GL): their ratios are others, up to
// 1.44 in FP64 and 1.6 in FP32, both at degree 2.  2D: facets take one tangential transform of a
// single line, so the nodal form's extra products buy nothing.
// What the dual form costs, sweeps on more than 10^3 cells against the nodal
// form's time: FP32 degree 1 1.37, 3 1.32, 6 1.15, 7 1.13, 8 1.22; FP64 degree 6
// 1.16, 7 1.13, 8 1.22.
template <typename T, int D, int N, bool VARK>
constexpr bool dual_sweep() {
  if (D == 2) return true;
  if (sizeof(T) == 2) return false;
  if (std::is_same<T, double>::value) return N > (VARK ? 8 : 6);
  return VARK || !(N == 3 || N == 5 || N == 6);
}
template <typename T, int D, int N, bool VARK>
constexpr bool dual_apply() {
  return D == 2 || VARK || !std::is_same<T, double>::value || N == 2 || N == 4;
}

// ---- dual form: lifts (also of the matrix-core sweep)

// r += SIGN x the dual lift of facets (k,0) and (k,1): value part at the
// facet node, normal derivative part along the line.
template <typename T, int D, int N, int SIGN>
__device__ __forceinline__ void dual_lifts(const DGArgs<T>& a, int cl, int k, int ln, const CT<T>* sNB,
                                               CT<T> (&r)[N]) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  const cptr<C> ep0 = as_const(a.ref) + RefOff<N>::EP0;
  const cptr<C> ep1 = as_const(a.ref) + RefOff<N>::EP1;
  const C* f0 = sNB + (cl * Sh::NF + 2 * k) * 2 * L;
  const C* f1 = f0 + 2 * L;
  const C v0 = f0[ln], d0 = f0[L + ln], v1 = f1[ln], d1 = f1[L + ln];
  constexpr C sg = C(SIGN);
  if (a.gl) {  // value functionals are dense (Gauss-Legendre nodes)
    const cptr<C> ev0 = as_const(a.ref) + RefOff<N>::EV0;
    const cptr<C> ev1 = as_const(a.ref) + RefOff<N>::EV1;
#pragma unroll
    for (int j = 0; j < N; ++j) r[j] += sg * (ev0[j] * v0 + ev1[j] * v1);
  } else {
    r[0] += sg * v0;
    r[N - 1] += sg * v1;
  }
#pragma unroll
  for (int j = 0; j < N; ++j) r[j] += sg * (ep0[j] * d0 + ep1[j] * d1);
}

// z_j of the Krylov projection (see DGArgs::kry), read by its storage type.
__device__ __forceinline__ double krylov_z(const DGArgs<double>& a, size_t i, double sc) {
  switch (a.zkind) {
    case 1: return (double)((const float*)a.zlow)[i] * sc;
    case 2: return (double)(float)((const _Float16*)a.zlow)[i] * sc;
    case 3: return (double)(float)((const __bf16*)a.zlow)[i] * sc;
    default: return ((const double*)a.zlow)[i] * sc;
  }
}

// Sum of v over the block, written by thread 0 to out (sh: one double per wave).
__device__ __forceinline__ void block_partial(double v, double* sh, double* out) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) sh[w] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < (int)((blockDim.x + 63) >> 6); ++i) s += sh[i];
    *out = s;
  }
}

// ---------------------------------------------------------------------------
// Bound and measurements of the nodal traversals: the LDS round trips between
// the axes and the trace traffic.  In dual form each facet field took two
// tangential transforms (24 N^3 multiply-adds per cell beside the volume's
// 6 N^4); in nodal form b takes Mhat^-1 along each axis (3 N^4, about half of
// that in even-odd form) and a facet field enters with one multiply-add per
// node, trace and facet.  Four instead of three waves per SIMD need no
// register cap (74 VGPRs at degree 4 in FP64, 125 before).  Measured sweep,
// dual -> nodal: FP64 Q4 32^3 57 -> 41.7 us, FP16 Q5 48^3 99 -> 82 us; FP64
// apply Q7 25^3 80 -> 55 us.
//
// Fused block-Jacobi sweep.  UZERO: u is identically zero on entry (first
// sweep of a coarse-level smoothing with zero initial guess): u and the
// neighbour traces are not read.  The thread's line of u stays in registers
// from the load to the update.
// LDS bytes of the sweep / apply bodies.
template <typename T, int D, int N, bool VARK, bool AD = false>
constexpr int cell_lds_bytes() {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  return (int)sizeof(C) * (Sh::CPB * Sh::NVP + Sh::CPB * Sh::NF * 2 * Sh::L + EigLDS<D, N, VARK, AD>::SIZE +
                           kappa_lds_entries<D, N, VARK>()) +
         (int)sizeof(int) * Sh::CPB;
}

// AD: adaptive mesh (neighbour traces by slot table, 16 class tables, per
// cell h scaling of b in 3D).
template <typename T, int D, int N, bool UZERO, bool VARK, bool IVAR = false, bool AD = false>
__device__ __forceinline__ void sweep_body(const DGArgs<T>& a, int bx, int by, char* lds) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  static_assert(D == 3, "nodal form: 3D");
  constexpr int L = Sh::L;
  constexpr int A = D - 1;  // axis of the thread's own line
  C* sNB = (C*)lds;  // pairs: first, for their alignment
  C* sW = sNB + Sh::CPB * Sh::NF * 2 * L;
  C* sE = sW + Sh::CPB * Sh::NVP;
  C* sKF = sE + EigLDS<D, N, VARK, AD>::SIZE;

  const Cells<D, N, AD> B(a, bx);
  const size_t rv = (size_t)by * a.vstride, rt = (size_t)by * a.tstride;
  int cl, ln;
  cell_line<D, N>(cl, ln);
  const bool act = B.valid(cl);
  const int c = B.cell(act ? cl : 0);
  const int mask = B.mask(a, act ? cl : 0, c);
  const int smask = IVAR ? 0 : mask;  // boundary classes of the block solve
  C hf = a.h_fwd;
  if constexpr (AD) {
    if (a.hscale) hf *= a.hscale[c];
  }
  auto get = [&](int k, C(&r)[N]) {
    const int base = lds_line<D, N>(cl, k, ln);
#pragma unroll
    for (int j = 0; j < N; ++j) r[j] = sW[base + j * lds_stride<D, N>(k)];
  };
  auto put = [&](int k, const C(&r)[N]) {
    const int base = lds_line<D, N>(cl, k, ln);
#pragma unroll
    for (int j = 0; j < N; ++j) sW[base + j * lds_stride<D, N>(k)] = r[j];
  };
  const size_t own = rv + (size_t)c * Sh::NV + ln;  // first node of the thread's line, stride L

  C ul[N], r[N], t[N];
  // the right-hand side in nodal form, when an earlier sweep has left it
  // (variable kappa, where the eigendata of the block solve fills the LDS pipe:
  // degree 5, 48^3, FP64, a smoothing call 2153 -> 2029 us.  With constant kappa the vector it
  // reads costs what the three contractions do: degree 4, 32^3, FP64 unchanged,
  // degree 2, 63^3, FP32 165 -> 170 us)
  constexpr bool BP = VARK && !UZERO && sizeof(T) == sizeof(C);
  const bool have = BP && a.bp_mode == 2;
  C* bp = a.bp + own;
  {
    const T* src = a.b + own;
    if constexpr (BP) src = have ? bp : src;
#pragma unroll
    for (int j = 0; j < N; ++j) r[j] = src[j * L];
  }
  if constexpr (!UZERO) {
#pragma unroll
    for (int j = 0; j < N; ++j) ul[j] = a.u_in[own + j * L];
  }
  stage_block<T, D, N, VARK, IVAR, AD, !UZERO, false, A>(a, a.tr_in + rt, B, cl, c, ln, act, mask, ul, sNB, sW, sE, sKF);
  if (have) hf = C(1);
#pragma unroll
  for (int j = 0; j < N; ++j) r[j] *= hf;

  // forward to the eigenvector basis along every axis; the last forward
  // axis also divides by the eigenvalue sums and transforms back
  auto middle = [&](int k) {
    C ls[N];
    eig_sums<D, N, VARK, IVAR, AD>(sE, cl, smask, k, ln, ls);
#pragma unroll
    for (int j = 0; j < N; ++j) t[j] *= recip(ls[j]);
    block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, k, t, r);
  };
  if constexpr (UZERO) {
    __syncthreads();  // eigendata staged
#pragma unroll
    for (int k = A; k >= 0; --k) {
      if (act) {
        if (k != A) get(k, r);
        block_mv<T, D, N, VARK, IVAR, AD, OP_ST>(a, sE, cl, smask, k, r, t);
        if (k == 0) {
          middle(0);
          put(0, r);
        } else {
          put(k, t);
        }
      }
      cell_sync<D, N>();
    }
    if (act) {
      get(1, r);
      block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, 1, r, t);
      put(1, t);
    }
    cell_sync<D, N>();
  } else {
    const cptr<C> Mi = as_const(a.ref) + RefOff<N>::MIC;
    if (have) {
      __syncthreads();  // traces staged, sW free
    } else {
      if constexpr (Cells<D, N, AD>::BR) __syncthreads();
      if (act) {
        cs_mv<N>(Mi, r);
        put(A, r);
      }
      if constexpr (Cells<D, N, AD>::BR)
        cell_sync<D, N>();
      else
        __syncthreads();  // traces staged
      if (act) {
        get(1, r);
        cs_mv<N>(Mi, r);
        put(1, r);
      }
      cell_sync<D, N>();
      // x: b in nodal values along every axis
      if (act) {
        get(0, r);
        cs_mv<N>(Mi, r);
        if (BP && a.bp_mode == 1) {
#pragma unroll
          for (int j = 0; j < N; ++j) bp[j * L] = r[j];
        }
      }
    }
    // minus the lifts
    if (act) {
      nodal_lifts<T, D, N, VARK, -1>(a, cl, 0, ln, sNB, sKF, r);
      block_mv<T, D, N, VARK, IVAR, AD, OP_SI>(a, sE, cl, smask, 0, r, t);
      put(0, t);
    }
    cell_sync<D, N>();
    if (act) {
      get(A, r);
      block_mv<T, D, N, VARK, IVAR, AD, OP_SI>(a, sE, cl, smask, A, r, t);
      put(A, t);
    }
    cell_sync<D, N>();
    if (act) {
      get(1, r);
      block_mv<T, D, N, VARK, IVAR, AD, OP_SI>(a, sE, cl, smask, 1, r, t);
      middle(1);
      put(1, r);
    }
    cell_sync<D, N>();
    if (act) {
      get(0, r);
      block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, 0, r, t);
      put(0, t);
    }
    cell_sync<D, N>();
  }
  // last inverse transform, update, store of u and of the traces
  T* trout = a.tr_out + rt;
  if (act) {
    get(A, r);
    block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, A, r, t);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const C uo0 = UZERO ? C(0) : ul[j];
      t[j] = (C(1) - a.omega) * uo0 + a.omega * t[j];
      a.u_out[own + j * L] = t[j];
    }
    put(A, t);
    store_line_traces<T, D, N, IVAR>(a, trout, B, cl, c, mask, A, ln, t);
  }
  cell_sync<D, N>();
  if (act) store_other_traces<T, D, N, A, IVAR>(a, trout, sW, B, cl, c, mask, ln);
}

// The sweep in dual form (see dual_sweep): S^T along every axis with the
// facet lifts, transformed along their tangential axes, subtracted before
// each; the x-lines of u and b stay in registers from load to update.
template <typename T, int D, int N, bool UZERO, bool VARK, bool IVAR = false, bool AD = false>
__device__ __forceinline__ void sweep_dual_body(const DGArgs<T>& a, int bx, int by, char* lds) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  C* sNB = (C*)lds;
  C* sW = sNB + Sh::CPB * Sh::NF * 2 * L;
  C* sE = sW + Sh::CPB * Sh::NVP;
  C* sKF = sE + EigLDS<D, N, VARK, AD>::SIZE;

  const Cells<D, N, AD> B(a, bx);
  const size_t rv = (size_t)by * a.vstride, rt = (size_t)by * a.tstride;
  int cl, ln;
  cell_line<D, N>(cl, ln);
  const bool act = B.valid(cl);
  const int c = B.cell(act ? cl : 0);
  const int base0 = line_base<D, N>(0, ln);
  const int mask = B.mask(a, act ? cl : 0, c);
  const int smask = IVAR ? 0 : mask;  // boundary classes of the block solve
  C hf = a.h_fwd;
  if constexpr (AD) {
    if (a.hscale) hf *= a.hscale[c];
  }

  C ul[N], bl[N];
  if (act) {
    const T* bs = a.b + rv + (size_t)c * Sh::NV + base0;
#pragma unroll
    for (int j = 0; j < N; ++j) bl[j] = bs[j];
    if (!UZERO) {
      const T* us = a.u_in + rv + (size_t)c * Sh::NV + base0;
#pragma unroll
      for (int j = 0; j < N; ++j) ul[j] = us[j];
    }
  }
  stage_block<T, D, N, VARK, IVAR, AD, !UZERO, true, 0>(a, a.tr_in + rt, B, cl, c, ln, act, mask, ul, sNB, sW, sE, sKF);
  if (act && ln == 0) mask_lds<D, N, VARK>(sKF)[cl] = mask;
  __syncthreads();
  if constexpr (!UZERO) {
#pragma unroll
    for (int pass = pass0_on_load<D, N, VARK, AD>() ? 1 : 0; pass < D - 1; ++pass) {
      facet_pass<T, D, N, VARK, IVAR, AD>(a, B, pass, sNB, sE, sKF);
      __syncthreads();
    }
  }

  // forward transforms S^T along x, y(, z) with the facet lifts subtracted
  // just before each axis is transformed
#pragma unroll
  for (int k = 0; k < D; ++k) {
    if (act) {
      const int base = lds_line<D, N>(cl, k, ln);
      C r[N], t[N];
      if (k == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = hf * bl[j];
      } else {
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = sW[base + j * lds_stride<D, N>(k)];
      }
      if (!UZERO) dual_lifts<T, D, N, -1>(a, cl, k, ln, sNB, r);
      block_mv<T, D, N, VARK, IVAR, AD, OP_ST>(a, sE, cl, smask, k, r, t);
      if (k == D - 1) {
        // diagonal scaling and the first inverse transform along the last axis
        C ls[N];
        eig_sums<D, N, VARK, IVAR, AD>(sE, cl, smask, k, ln, ls);
#pragma unroll
        for (int j = 0; j < N; ++j) t[j] *= recip(ls[j]);
        block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, k, t, r);
#pragma unroll
        for (int j = 0; j < N; ++j) t[j] = r[j];
      }
#pragma unroll
      for (int j = 0; j < N; ++j) sW[base + j * lds_stride<D, N>(k)] = t[j];
    }
    __syncthreads();
  }
  // inverse transforms S along the remaining axes; the last one is fused
  // with the update, the store of u and of the x-facet traces
  T* trout = a.tr_out + rt;
#pragma unroll
  for (int k = D - 2; k >= 0; --k) {
    if (act) {
      const int base = lds_line<D, N>(cl, k, ln);
      C r[N], t[N];
#pragma unroll
      for (int j = 0; j < N; ++j) r[j] = sW[base + j * lds_stride<D, N>(k)];
      block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, k, r, t);
      if (k == 0) {
        T* uo = a.u_out + rv + (size_t)c * Sh::NV + base0;
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const C uo0 = UZERO ? C(0) : ul[j];
          t[j] = (C(1) - a.omega) * uo0 + a.omega * t[j];
          sW[base + j] = t[j];
          uo[j] = t[j];
        }
        store_line_traces<T, D, N, IVAR>(a, trout, B, cl, c, mask, 0, ln, t);
      } else {
#pragma unroll
        for (int j = 0; j < N; ++j) sW[base + j * lds_stride<D, N>(k)] = t[j];
      }
    }
    __syncthreads();
  }
  if (act) store_other_traces<T, D, N, 0, IVAR>(a, trout, sW, B, cl, c, mask, ln);
}

// ---------------------------------------------------------------------------
// Per-cell fast-diagonalisation data of a variable-coefficient level, built
// on the device at setup with the eigensolve of recompute_eig (FP64): for
// every cell and axis the record S (N^2) | lambda (N) of L_k S = Mhat S
// diag(lambda), S^T Mhat S = I, in the layout the stored-eigendata kernels
// read ([cell][axis][S | lambda]).  a.rk holds [Khat | C^-1], a.kappa the
// per-cell kappa; a.out receives the records, a.flag is set to 1 if an
// eigenvalue is not positive and finite (the cell block is not positive
// definite).
template <typename C, int D, int N>
constexpr int build_eig_lds_bytes() {
  return (int)sizeof(C) *
         (EigLDS<D, N, true>::SIZE + kappa_lds_entries<D, N, true>() + DGShape<D, N>::CPB * D * N * N);  // scratch
}
template <typename C, int D, int N>
__global__ __launch_bounds__((DGShape<D, N>::BLOCK)) void k_build_eig(DGArgs<C> a) {
  using Sh = DGShape<D, N>;
  constexpr int NN = N * N;
  __shared__ __attribute__((aligned(16))) char lds[build_eig_lds_bytes<C, D, N>()];
  C* sE = (C*)lds;
  C* sKF = sE + EigLDS<D, N, true>::SIZE;
  int id, rhs;
  block_of_grid<D, N, false>(a, id, rhs);
  const Cells<D, N, false> B(a, id);
  load_eig<C, D, N, true>(a, B, sE, sKF);
  __syncthreads();
  recompute_eig<C, D, N>(a, B.count(), sE, sKF, sKF + kappa_lds_entries<D, N, true>());
  __syncthreads();
  constexpr int R = D * (NN + N);  // words per cell
  bool bad = false;
  for (int i = work_tid<D, N>(); i < B.count() * R; i += Sh::NT) {
    if (!B.valid(i / R)) continue;
    const C v = sE[i];
    a.out[(size_t)B.cell(i / R) * R + i % R] = v;
    if (i % (NN + N) >= NN && !(v > C(0) && v < C(1e30))) bad = true;
  }
  if (bad && a.flag) atomicOr(a.flag, 1);
}

// ---------------------------------------------------------------------------
// Volume contractions of the 16-bit storage sweep on the matrix cores.
//
// One contraction stage replaces every line along axis k of the block's
// cells (FP32, in sW) by G_cell x line, with G = S^T (TR) or S of the cell's
// axis-k record.  A 16x16x16 product D = A B holds NB = 16/N cells on the
// block diagonal of A = diag(G_c0, .., G_c(NB-1)) (zero padded) and 16 lines
// of each of those cells as the columns of B (row N kb + j of B: node j of
// the line in cell kb), so that D row N rb + i, column c is node i of line c
// of cell rb.  The operands are rounded to the storage format (FP16 or BF16)
// and the products accumulate in FP32.  Operand lane layout (16x16x16):
// lane l holds A[l%16][4(l/16)+j], B[4(l/16)+j][l%16] and D[4(l/16)+j][l%16],
// j = 0..3.  SCALE multiplies the result by 1 / (lambda sum) of the node
// (the diagonal of the fast-diagonalised block inverse, applied after S^T
// along the last axis).  Called by every thread of the block (whole waves);
// the products of a wave cover disjoint lines.
typedef _Float16 mf_half4 __attribute__((ext_vector_type(4)));
typedef short mf_short4 __attribute__((ext_vector_type(4)));
typedef float mf_float4 __attribute__((ext_vector_type(4)));

template <typename T>
struct Mfma16;
template <>
struct Mfma16<_Float16> {
  static __device__ __forceinline__ mf_float4 mul(const float (&a)[4], const float (&b)[4]) {
    mf_half4 x, y;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = (_Float16)a[j];
      y[j] = (_Float16)b[j];
    }
    const mf_float4 z = {0.f, 0.f, 0.f, 0.f};
    return __builtin_amdgcn_mfma_f32_16x16x16f16(x, y, z, 0, 0, 0);
  }
};
template <>
struct Mfma16<__bf16> {
  static __device__ __forceinline__ mf_float4 mul(const float (&a)[4], const float (&b)[4]) {
    mf_short4 x, y;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = __builtin_bit_cast(short, (__bf16)a[j]);
      y[j] = __builtin_bit_cast(short, (__bf16)b[j]);
    }
    const mf_float4 z = {0.f, 0.f, 0.f, 0.f};
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(x, y, z, 0, 0, 0);
  }
};

template <typename T, int D, int N, bool VARK, bool IVAR, bool TR, bool SCALE>
__device__ __forceinline__ void mfma_stage(float* sW, const float* sE, const int* sMask, int nc, int k) {
  using Sh = DGShape<D, N>;
  constexpr int NN = N * N;
  constexpr int L = Sh::L;
  constexpr int NB = 16 / N;               // cells per product
  constexpr int CH = (L + 15) / 16;        // 16-line chunks per cell
  constexpr int TASKS = (Sh::CPB + NB - 1) / NB * CH;
  constexpr int NW = Sh::BLOCK / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = lane & 15, kq = lane >> 4;
  const int stride = lds_stride<D, N>(k);
  // cell record of block-diagonal block b (clamped to a staged cell)
  auto rec = [&](int cl) -> const float* {
    if constexpr (VARK)
      return sE + (cl * D + k) * Sh::EGV;
    else
      return sE + (IVAR ? 0 : axis_class(sMask[cl], k)) * Sh::EGS;
  };
  for (int t = wave; t < TASKS; t += NW) {  // uniform over the wave
    const int g = t / CH, q = t % CH;
    const int line = 16 * q + c;
    const int lc = min(line, L - 1);
    const int lb = lds_line<D, N>(0, k, lc);
    float av[4], bv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kk = 4 * kq + j;
      const int kb = kk / N, jj = kk % N;
      const int cl = g * NB + kb;
      const bool okb = kb < NB && cl < nc && line < L;
      const float x = sW[min(cl, nc - 1) * Sh::NVP + lb + (jj < N ? jj : 0) * stride];
      bv[j] = okb ? x : 0.f;
      const int rb = c / N, ii = c % N;
      const int cla = g * NB + rb;
      const bool oka = rb == kb && rb < NB && cla < nc;
      const float* G = rec(min(cla, nc - 1));
      const float gv = TR ? G[jj * N + ii] : G[ii * N + jj];
      av[j] = oka ? gv : 0.f;
    }
    const mf_float4 d = Mfma16<T>::mul(av, bv);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int i = 4 * kq + j;
      const int rb = i / N, ii = i % N;
      const int cl = g * NB + rb;
      if (rb < NB && cl < nc && line < L) {
        float v = d[j];
        if constexpr (SCALE) {
          // lambda sum of node (line, ii) along the last axis k = D - 1
          const int clc = cl;
          constexpr int LO = VARK ? NN : 2 * NN;  // lambda within the record
          float ls;
          if constexpr (D == 2) {
            const float* E0 = VARK ? sE + (clc * D + 0) * Sh::EGV : sE + (IVAR ? 0 : axis_class(sMask[clc], 0)) * Sh::EGS;
            const float* E1 = VARK ? sE + (clc * D + 1) * Sh::EGV : sE + (IVAR ? 0 : axis_class(sMask[clc], 1)) * Sh::EGS;
            ls = E0[LO + line] + E1[LO + ii];
          } else {
            const float* E0 = VARK ? sE + (clc * D + 0) * Sh::EGV : sE + (IVAR ? 0 : axis_class(sMask[clc], 0)) * Sh::EGS;
            const float* E1 = VARK ? sE + (clc * D + 1) * Sh::EGV : sE + (IVAR ? 0 : axis_class(sMask[clc], 1)) * Sh::EGS;
            const float* E2 = VARK ? sE + (clc * D + 2) * Sh::EGV : sE + (IVAR ? 0 : axis_class(sMask[clc], 2)) * Sh::EGS;
            ls = E0[LO + line % N] + E1[LO + line / N] + E2[LO + ii];
          }
          v *= recip(ls);
        }
        sW[cl * Sh::NVP + lb + ii * stride] = v;
      }
    }
  }
}

// Fused sweep of a 16-bit storage type with the volume contractions on the
// matrix cores (mfma_stage); facet flux fields, lifts, update and traces as
// in dual form (facet_pass, dual_lifts).  Launched with whole waves (DGShape::BLOCK threads).
template <typename T, int D, int N, bool UZERO, bool VARK, bool IVAR>
__device__ __forceinline__ void sweep_body_mfma(const DGArgs<T>& a, int bx, int by, char* lds) {
  using C = CT<T>;
  static_assert(sizeof(C) == 4, "matrix-core sweep: 16-bit storage, FP32 compute");
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  C* sNB = (C*)lds;  // pairs: first, for their alignment
  C* sW = sNB + Sh::CPB * Sh::NF * 2 * L;
  C* sE = sW + Sh::CPB * Sh::NVP;
  C* sKF = sE + EigLDS<D, N, VARK>::SIZE;
  int* sMask = mask_lds<D, N, VARK>(sKF);

  const Cells<D, N, false> B(a, bx);
  const size_t rv = (size_t)by * a.vstride, rt = (size_t)by * a.tstride;
  int cl, ln;
  cell_line<D, N>(cl, ln);
  const bool act = B.valid(cl);
  const int c = B.cell(act ? cl : 0);
  const int base0 = line_base<D, N>(0, ln);
  const int mask = B.mask(a, act ? cl : 0, c);

  C ul[N], bl[N];
  if (act) {
    const T* bs = a.b + rv + (size_t)c * Sh::NV + base0;
#pragma unroll
    for (int j = 0; j < N; ++j) bl[j] = bs[j];
    if (!UZERO) {
      const T* us = a.u_in + rv + (size_t)c * Sh::NV + base0;
#pragma unroll
      for (int j = 0; j < N; ++j) ul[j] = us[j];
    }
  }
  static_assert(!Cells<D, N, false>::BR, "16-bit storage: runs of cells");
  if (act && ln == 0) sMask[cl] = mask;
  stage_block<T, D, N, VARK, IVAR, false, !UZERO, true, 0>(a, a.tr_in + rt, B, cl, c, ln, act, mask, ul, sNB, sW, sE, sKF);
  __syncthreads();
  if constexpr (!UZERO) {
#pragma unroll
    for (int pass = pass0_on_load<D, N, VARK, false>() ? 1 : 0; pass < D - 1; ++pass) {
      facet_pass<T, D, N, VARK, IVAR>(a, B, pass, sNB, sE, sKF);
      __syncthreads();
    }
  }
  // forward: right-hand side minus the facet lifts along each axis (vector
  // units, one thread per line), then S^T along that axis on the matrix
  // cores; the last forward stage applies the diagonal scaling
#pragma unroll
  for (int k = 0; k < D; ++k) {
    if (act && (k == 0 || !UZERO)) {
      const int base = lds_line<D, N>(cl, k, ln);
      C r[N];
      if (k == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = a.h_fwd * bl[j];
      } else {
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = sW[base + j * lds_stride<D, N>(k)];
      }
      if (!UZERO) dual_lifts<T, D, N, -1>(a, cl, k, ln, sNB, r);
#pragma unroll
      for (int j = 0; j < N; ++j) sW[base + j * lds_stride<D, N>(k)] = r[j];
    }
    __syncthreads();
    if (k == D - 1)
      mfma_stage<T, D, N, VARK, IVAR, true, true>(sW, sE, sMask, B.nc, k);
    else
      mfma_stage<T, D, N, VARK, IVAR, true, false>(sW, sE, sMask, B.nc, k);
    __syncthreads();
  }
  // inverse: S along every axis, last axis first
#pragma unroll
  for (int k = D - 1; k >= 0; --k) {
    mfma_stage<T, D, N, VARK, IVAR, false, false>(sW, sE, sMask, B.nc, k);
    __syncthreads();
  }
  // update, store of u and of the traces
  T* trout = a.tr_out + rt;
  if (act) {
    T* uo = a.u_out + rv + (size_t)c * Sh::NV + base0;
    C t[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const C uo0 = UZERO ? C(0) : ul[j];
      t[j] = (C(1) - a.omega) * uo0 + a.omega * sW[lds_line<D, N>(cl, 0, ln) + j];
      sW[lds_line<D, N>(cl, 0, ln) + j] = t[j];
      uo[j] = t[j];
    }
    store_line_traces<T, D, N, IVAR>(a, trout, B, cl, c, mask, 0, ln, t);
  }
  __syncthreads();
  if (act) store_other_traces<T, D, N, 0, IVAR>(a, trout, sW, B, cl, c, mask, ln);
}

// The sweep of a block in its form.  UZERO: the forms differ in the axes' order
// alone.
template <typename T, int D, int N, bool UZERO, bool VARK, bool IVAR = false, bool AD = false, bool GL = false>
__device__ __forceinline__ void sweep_cells(const DGArgs<T>& a, int bx, int by, char* lds) {
  if constexpr (D == 2 || (!UZERO && (GL || dual_sweep<T, D, N, VARK>())))
    sweep_dual_body<T, D, N, UZERO, VARK, IVAR, AD>(a, bx, by, lds);
  else
    sweep_body<T, D, N, UZERO, VARK, IVAR, AD>(a, bx, by, lds);
}

// Waves per SIMD asked of the sweep: as many as its LDS allows (160 KB per
// CU), so that the compiler does not spend registers on reading ahead past
// that occupancy.  Variable kappa and plain products (block_mv, eo) keep whole 1D
// matrices in registers: two waves at degree 7 and 8 (left to itself the
// compiler reaches one), no bound below.
template <typename T, int D, int N, bool VARK>
constexpr int sweep_waves_per_eu() {
  if (D != 3 || sizeof(CT<T>) != 8) return 1;
  if (VARK || (HPMG_TILE == 3 && N > 6)) return N >= 8 ? 2 : 1;
  constexpr int blocks = 160 * 1024 / cell_lds_bytes<T, D, N, false>();
  constexpr int waves = blocks * (DGShape<D, N>::BLOCK / 64) / 4;
  return waves < 5 ? waves : 5;
}
template <typename T, int D, int N, bool UZERO, bool VARK, bool IVAR, bool MF = false, bool AD = false, bool GL = false>
__global__ __launch_bounds__((DGShape<D, N>::BLOCK))
__attribute__((amdgpu_waves_per_eu(sweep_waves_per_eu<T, D, N, VARK>()))) void k_sweep(DGArgs<T> a) {
  __shared__ __attribute__((aligned(16))) char lds[cell_lds_bytes<T, D, N, VARK, AD>()];
  int id, rhs;
  block_of_grid<D, N, AD>(a, id, rhs);
  if constexpr (MF)
    sweep_body_mfma<T, D, N, UZERO, VARK, IVAR>(a, id, rhs, lds);
  else
    sweep_cells<T, D, N, UZERO, VARK, IVAR, AD, GL>(a, id, rhs, lds);
}

// ---------------------------------------------------------------------------
// Restriction (E^T)^(x d) of the cell residuals in sW, one axis per pass,
// through sNB (every lift has been read) into a.out: a coarse DG cell
// vector, or the 2^d Q1 corner contributions of each cell.
template <typename T, int D, int N, int NC, bool AD>
__device__ __forceinline__ void restrict_body(const DGArgs<T>& a, const Cells<D, N, AD>& B, int by, CT<T>* sNB,
                                              CT<T>* sW) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  const int tid = work_tid<D, N>();
  const int nc = B.count();
  // NC < 0: the coarse node count ncr comes at run time (a.ncd <= N), loops
  // run to N.
  constexpr int NCB = NC > 0 ? NC : N;
  const int ncr = NC > 0 ? NC : a.ncd;
  const cptr<C> E = as_const(a.ref) + RefOff<N>::E;
  const int NCD = (D == 2) ? ncr * ncr : ncr * ncr * ncr;
  constexpr int NBS = Sh::NF * 2 * L;  // per-cell stride of sNB
  C* out = a.out + (size_t)by * a.cstride;
  // x: sW[cl][..][a] -> sNB[cl][ln][a'] (a' + ncr*ln)
  for (int i = tid; i < nc * L; i += Sh::NT) {
    const int c2 = i / L, l2 = i % L;
    C x[N];
#pragma unroll
    for (int j = 0; j < N; ++j) x[j] = sW[lds_line<D, N>(c2, 0, l2) + j];
#pragma unroll
    for (int jc = 0; jc < NCB; ++jc) {
      if (jc < ncr) {
        C s = 0;
#pragma unroll
        for (int j = 0; j < N; ++j) s += E[j * ncr + jc] * x[j];
        sNB[c2 * NBS + jc + ncr * l2] = s;
      }
    }
  }
  __syncthreads();
  if constexpr (D == 2) {
    // y: sNB[cl][b][a'] -> dst[a' + ncr b']
    for (int i = tid; i < nc * ncr; i += Sh::NT) {
      const int c2 = i / ncr, ac = i % ncr;
      C* dst = out + (size_t)B.cell(c2) * NCD;
      C x[N];
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = sNB[c2 * NBS + ac + ncr * j];
#pragma unroll
      for (int bc = 0; bc < NCB; ++bc) {
        if (bc < ncr) {
          C s = 0;
#pragma unroll
          for (int j = 0; j < N; ++j) s += E[j * ncr + bc] * x[j];
          dst[ac + ncr * bc] = s;
        }
      }
    }
  } else {
    // y: sNB[cl][c][b][a'] (a' + ncr(b + N c)) -> sW[cl][c][b'][a'] (a' + ncr(b' + ncr c))
    for (int i = tid; i < nc * ncr * N; i += Sh::NT) {
      const int c2 = i / (ncr * N), rem = i % (ncr * N);
      const int ac = rem % ncr, cz = rem / ncr;
      C x[N];
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = sNB[c2 * NBS + ac + ncr * (j + N * cz)];
#pragma unroll
      for (int bc = 0; bc < NCB; ++bc) {
        if (bc < ncr) {
          C s = 0;
#pragma unroll
          for (int j = 0; j < N; ++j) s += E[j * ncr + bc] * x[j];
          sW[c2 * Sh::NV + ac + ncr * (bc + ncr * cz)] = s;
        }
      }
    }
    __syncthreads();
    // z: sW[cl][c][b'][a'] -> dst[a' + ncr b' + ncr^2 c']
    for (int i = tid; i < nc * ncr * ncr; i += Sh::NT) {
      const int c2 = i / (ncr * ncr), rem = i % (ncr * ncr);
      if (!B.valid(c2)) continue;
      C* dst = out + (size_t)B.cell(c2) * NCD;
      C x[N];
#pragma unroll
      for (int j = 0; j < N; ++j) x[j] = sW[c2 * Sh::NV + rem + ncr * ncr * j];
#pragma unroll
      for (int ccz = 0; ccz < NCB; ++ccz) {
        if (ccz < ncr) {
          C s = 0;
#pragma unroll
          for (int j = 0; j < N; ++j) s += E[j * ncr + ccz] * x[j];
          dst[rem + ncr * ncr * ccz] = s;
        }
      }
    }
  }
}

// The block's share of p.(A p) in the outer FP64 iteration (kdot).
template <typename T, int NC, bool RESID>
__device__ __forceinline__ void apply_partial(const DGArgs<T>& a, double pdot, int block) {
  if constexpr (std::is_same<T, double>::value && NC == 0 && !RESID) {
    if (a.kdot) {
      __shared__ double sh[16];
      block_partial(pdot, sh, a.kpartial + block);
    }
  }
}

// apply_body in dual form: Si along every axis, the eigenvalue sums, Si^T
// back, with the facet lifts transformed along their tangential axes
// (facet_pass) and added right after each axis.  See dual_apply for where it
// is used.
template <typename T, int D, int N, int NC, bool RESID, bool VARK, bool IVAR = false, bool AD = false>
__device__ __forceinline__ void apply_dual_body(const DGArgs<T>& a, int bx, int by, char* lds) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  C* sNB = (C*)lds;  // as in sweep_body
  C* sW = sNB + Sh::CPB * Sh::NF * 2 * L;
  C* sE = sW + Sh::CPB * Sh::NVP;
  C* sKF = sE + EigLDS<D, N, VARK, AD>::SIZE;

  const Cells<D, N, AD> B(a, bx);
  const size_t rv = (size_t)by * a.vstride, rt = (size_t)by * a.tstride;
  int cl, ln;
  cell_line<D, N>(cl, ln);
  const bool act = B.valid(cl);
  const int c = B.cell(act ? cl : 0);
  const int base0 = line_base<D, N>(0, ln);
  const int mask = B.mask(a, act ? cl : 0, c);
  const int smask = IVAR ? 0 : mask;  // boundary classes of the block solve
  C ha = a.h_apply;
  if constexpr (AD) {
    if (a.hscale) ha /= a.hscale[c];
  }

  C ul[N], bl[N];
  if (act) {
    const T* us = a.u_in + rv + (size_t)c * Sh::NV + base0;
#pragma unroll
    for (int j = 0; j < N; ++j) ul[j] = us[j];
    if constexpr (RESID) {
      const T* bs = a.b + rv + (size_t)c * Sh::NV + base0;
#pragma unroll
      for (int j = 0; j < N; ++j) bl[j] = bs[j];
    }
  }
  double pdot = 0.0;  // share of p.(A p) (kdot)
  stage_block<T, D, N, VARK, IVAR, AD, true, true, 0, true>(a, a.tr_in + rt, B, cl, c, ln, act, mask, ul, sNB, sW, sE, sKF);
  if (act && ln == 0) mask_lds<D, N, VARK>(sKF)[cl] = mask;
  __syncthreads();
#pragma unroll
  for (int pass = pass0_on_load<D, N, VARK, AD>() ? 1 : 0; pass < D - 1; ++pass) {
    facet_pass<T, D, N, VARK, IVAR, AD, true>(a, B, pass, sNB, sE, sKF);
    __syncthreads();
  }

  // Si along every axis, diagonal scaling, then Si^T (= M S) back with the
  // lifts added right after each axis is transformed back.
#pragma unroll
  for (int k = 0; k < D; ++k) {
    if (act) {
      const int base = lds_line<D, N>(cl, k, ln);
      C r[N], t[N];
      if (k == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = ul[j];
      } else {
#pragma unroll
        for (int j = 0; j < N; ++j) r[j] = sW[base + j * lds_stride<D, N>(k)];
      }
      block_mv<T, D, N, VARK, IVAR, AD, OP_SI, true>(a, sE, cl, smask, k, r, t);
      if (k == D - 1) {
        C ls[N];
        eig_sums<D, N, VARK, IVAR, AD>(sE, cl, smask, k, ln, ls);
#pragma unroll
        for (int j = 0; j < N; ++j) t[j] *= ls[j];
        block_mv<T, D, N, VARK, IVAR, AD, OP_SIT, true>(a, sE, cl, smask, k, t, r);
        dual_lifts<T, D, N, 1>(a, cl, k, ln, sNB, r);
#pragma unroll
        for (int j = 0; j < N; ++j) t[j] = r[j];
      }
#pragma unroll
      for (int j = 0; j < N; ++j) sW[base + j * lds_stride<D, N>(k)] = t[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int k = D - 2; k >= 0; --k) {
    if (act) {
      const int base = lds_line<D, N>(cl, k, ln);
      C r[N], t[N];
#pragma unroll
      for (int j = 0; j < N; ++j) r[j] = sW[base + j * lds_stride<D, N>(k)];
      block_mv<T, D, N, VARK, IVAR, AD, OP_SIT, true>(a, sE, cl, smask, k, r, t);
      dual_lifts<T, D, N, 1>(a, cl, k, ln, sNB, t);
      if (k == 0) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
          t[j] *= ha;
          if constexpr (RESID) t[j] = bl[j] - t[j];
          if constexpr (NC == 0)
            a.out[rv + (size_t)c * Sh::NV + base0 + j] = t[j];
          else
            sW[base + j] = t[j];
          if constexpr (std::is_same<T, double>::value && NC == 0 && !RESID) pdot += ul[j] * t[j];
        }
      } else {
#pragma unroll
        for (int j = 0; j < N; ++j) sW[base + j * lds_stride<D, N>(k)] = t[j];
      }
    }
    __syncthreads();
  }
  apply_partial<T, NC, RESID>(a, pdot, B.number(bx));
  if constexpr (NC != 0) restrict_body<T, D, N, NC>(a, B, by, sNB, sW);
}

// y = A u (RESID: r = b - A u), optionally restricted to the next coarser
// level: NC > 0 gives per cell (E^C x E^C x E^C) r with E the interpolation
// from the coarse nodes (DG_q: a coarse cell vector; Q1: the 2^d corner
// contributions of each cell, summed over cells by the gather kernel).
// Needs the traces of u in tr_in.
template <typename T, int D, int N, int NC, bool RESID, bool VARK, bool IVAR = false, bool AD = false>
__device__ __forceinline__ void apply_body(const DGArgs<T>& a, int bx, int by, char* lds) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  static_assert(D == 3, "nodal form: 3D");
  constexpr int L = Sh::L;
  constexpr int A = D - 1;  // axis of the thread's own line
  C* sNB = (C*)lds;  // pairs: first, for their alignment
  C* sW = sNB + Sh::CPB * Sh::NF * 2 * L;
  C* sE = sW + Sh::CPB * Sh::NVP;
  C* sKF = sE + EigLDS<D, N, VARK, AD>::SIZE;

  const Cells<D, N, AD> B(a, bx);
  const size_t rv = (size_t)by * a.vstride, rt = (size_t)by * a.tstride;
  int cl, ln;
  cell_line<D, N>(cl, ln);
  const bool act = B.valid(cl);
  const int c = B.cell(act ? cl : 0);
  const int mask = B.mask(a, act ? cl : 0, c);
  const int smask = IVAR ? 0 : mask;  // boundary classes of the block solve
  C ha = a.h_apply;
  if constexpr (AD) {
    if (a.hscale) ha /= a.hscale[c];
  }

  auto get = [&](int k, C(&r)[N]) {
    const int base = lds_line<D, N>(cl, k, ln);
#pragma unroll
    for (int j = 0; j < N; ++j) r[j] = sW[base + j * lds_stride<D, N>(k)];
  };
  auto put = [&](int k, const C(&r)[N]) {
    const int base = lds_line<D, N>(cl, k, ln);
#pragma unroll
    for (int j = 0; j < N; ++j) sW[base + j * lds_stride<D, N>(k)] = r[j];
  };
  const size_t own = rv + (size_t)c * Sh::NV + ln;  // first node of the thread's line, stride L

  C ul[N], bl[N], r[N], t[N];
#pragma unroll
  for (int j = 0; j < N; ++j) ul[j] = a.u_in[own + j * L];
  if constexpr (RESID) {
#pragma unroll
    for (int j = 0; j < N; ++j) bl[j] = a.b[own + j * L];
  }
  stage_block<T, D, N, VARK, IVAR, AD, true, false, A>(a, a.tr_in + rt, B, cl, c, ln, act, mask, ul, sNB, sW, sE, sKF);
  __syncthreads();
  double pdot = 0.0;  // share of p.(A p) (kdot)

  // S Lambda Si u: nodal values of Mhat^-1 (A_{K<-K} u) along every axis
#pragma unroll
  for (int k = A; k >= 0; --k) {
    if (act) {
      if (k == A) {
        block_mv<T, D, N, VARK, IVAR, AD, OP_SI>(a, sE, cl, smask, k, ul, t);
      } else {
        get(k, r);
        block_mv<T, D, N, VARK, IVAR, AD, OP_SI>(a, sE, cl, smask, k, r, t);
      }
      if (k == 0) {
        C ls[N];
        eig_sums<D, N, VARK, IVAR, AD>(sE, cl, smask, 0, ln, ls);
#pragma unroll
        for (int j = 0; j < N; ++j) t[j] *= ls[j];
        block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, 0, t, r);
        put(0, r);
      } else {
        put(k, t);
      }
    }
    cell_sync<D, N>();
  }
  if (act) {
    get(A, r);
    block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, A, r, t);
    put(A, t);
  }
  cell_sync<D, N>();
  // plus the lifts (in the y-lines), times the mass along every axis
  const cptr<C> Mc = as_const(a.ref) + RefOff<N>::MC;
  if (act) {
    get(1, r);
    block_mv<T, D, N, VARK, IVAR, AD, OP_S>(a, sE, cl, smask, 1, r, t);
    nodal_lifts<T, D, N, VARK, 1>(a, cl, 1, ln, sNB, sKF, t);
    cs_mv<N>(Mc, t);
    put(1, t);
  }
  cell_sync<D, N>();
  if (act) {
    get(0, r);
    cs_mv<N>(Mc, r);
    put(0, r);
  }
  cell_sync<D, N>();
  if (act) {
    get(A, t);
    cs_mv<N>(Mc, t);
#pragma unroll
    for (int j = 0; j < N; ++j) {
      t[j] *= ha;
      if (RESID) t[j] = bl[j] - t[j];
    }
    if constexpr (NC == 0) {
#pragma unroll
      for (int j = 0; j < N; ++j) a.out[own + j * L] = t[j];
      if constexpr (std::is_same<T, double>::value && !RESID) {
#pragma unroll
        for (int j = 0; j < N; ++j) pdot += ul[j] * t[j];
      }
    } else {
      put(A, t);
    }
  }
  if constexpr (NC != 0) __syncthreads();
  apply_partial<T, NC, RESID>(a, pdot, B.number(bx));
  if constexpr (NC != 0) restrict_body<T, D, N, NC>(a, B, by, sNB, sW);
}

template <typename T, int D, int N, int NC, bool RESID, bool VARK, bool IVAR = false, bool AD = false, bool GL = false>
__device__ __forceinline__ void apply_cells(const DGArgs<T>& a, int bx, int by, char* lds) {
  if constexpr (GL || dual_apply<T, D, N, VARK>())
    apply_dual_body<T, D, N, NC, RESID, VARK, IVAR, AD>(a, bx, by, lds);
  else
    apply_body<T, D, N, NC, RESID, VARK, IVAR, AD>(a, bx, by, lds);
}

// Apply holds u, b and the neighbour traces in registers at once; for the
// FP64 degree-4 instances at most 128 VGPRs (four waves per SIMD, no spills).
template <typename T, int N>
constexpr int apply_waves_per_eu() {
  return (sizeof(T) == 8 && N <= 5) ? 4 : 1;
}
template <typename T, int D, int N, int NC, bool RESID, bool VARK, bool IVAR, bool AD = false, bool GL = false>
__global__ __launch_bounds__((DGShape<D, N>::BLOCK))
__attribute__((amdgpu_waves_per_eu(apply_waves_per_eu<T, N>()))) void k_apply(DGArgs<T> a) {
  __shared__ __attribute__((aligned(16))) char lds[cell_lds_bytes<T, D, N, VARK, AD>()];
  int id, rhs;
  block_of_grid<D, N, AD>(a, id, rhs);
  apply_cells<T, D, N, NC, RESID, VARK, IVAR, AD, GL>(a, id, rhs, lds);
}

// ---------------------------------------------------------------------------
// u += P e (NC > 0; DG_q cell vector or Q1 vertex vector) and projection of
// u onto the facet traces (NC = 0: projection only, the warm-up traversal of
// Algorithm BlockJacobi; NC > 0: fused prolongation + projection,
// Section 5.1.1).
template <typename T, int D, int N, int NC>
constexpr int prolong_lds_bytes() {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  return (int)sizeof(C) * (Sh::CPB * Sh::NVP + (NC != 0 ? Sh::CPB * Sh::NV + Sh::CPB * Sh::NF * 2 * Sh::L : 0));
}

template <typename T, int D, int N, int NC, bool IVAR = false, bool AD = false>
__device__ __forceinline__ void prolong_body(const DGArgs<T>& a, int bx, int by, char* lds) {
  using C = CT<T>;
  using Sh = DGShape<D, N>;
  constexpr int L = Sh::L;
  C* sU = (C*)lds;
  C* sW = sU + Sh::CPB * Sh::NVP;
  C* sNB = sW + Sh::CPB * Sh::NV;

  const Cells<D, N, AD> B(a, bx);
  const size_t rv = (size_t)by * a.vstride, rt = (size_t)by * a.tstride;
  const int tid = work_tid<D, N>();
  int cl, ln;
  cell_line<D, N>(cl, ln);
  const bool act = B.valid(cl);
  const int c = B.cell(act ? cl : 0);
  const int mask = B.mask(a, act ? cl : 0, c);
  const int nc = B.count();
  // NC < 0: coarse node count ncr at run time (a.ncd <= N); loops run to
  // NCB = N with the entries past ncr skipped
  constexpr int NCB = NC > 0 ? NC : (NC < 0 ? N : 1);
  const int ncr = NC >= 0 ? NC : a.ncd;
  const int NCD = (NC == 0) ? 0 : ((D == 2) ? ncr * ncr : ncr * ncr * ncr);

  // the thread's own line: along the last axis in 3D (as in the nodal
  // traversals), along x in 2D (as in the dual ones)
  constexpr int F = D == 3 ? 2 : 0, ST = line_stride<N>(F);
  const int lb = line_base<D, N>(F, ln);
  C u[N];
  const size_t own = rv + (size_t)c * Sh::NV + lb;
#pragma unroll
  for (int j = 0; j < N; ++j) u[j] = a.u_in[own + j * ST];
  if constexpr (std::is_same<T, double>::value && NC == 0) {
    if (a.kry && act) {  // p = z + beta p, in place
      const double beta = a.kscal[3];
      const double sc = a.zscaled ? a.kscal[8] / a.kmul : 1.0;
#pragma unroll
      for (int j = 0; j < N; ++j) {
        const double zj = krylov_z(a, own + j * ST, sc);
        u[j] = beta == 0.0 ? zj : zj + beta * u[j];
      }
#pragma unroll
      for (int j = 0; j < N; ++j) a.u_out[own + j * ST] = u[j];
    }
  }
  if constexpr (NC != 0) {
    const C* cs = a.coarse + (size_t)by * a.cstride;
    if (a.coarse_cg != 1) {
      // a coarse DG cell vector, or the Q1 corner values of every cell
      for (int i = tid; i < nc * NCD; i += Sh::NT)
        sW[(i / NCD) * Sh::NV + i % NCD] = cs[(size_t)B.cell(i / NCD) * NCD + i % NCD];
    } else {
      // Q1 corner values of each cell from the interior-vertex vector
      const int nv = a.n - 1;
      for (int i = tid; i < nc * NCD; i += Sh::NT) {
        const int c2 = i / NCD, corner = i % NCD;
        const int cc = B.cell(c2);
        int x[3];
        x[0] = cc % a.n;
        const int rr = cc / a.n;
        x[1] = (D == 2) ? rr : rr % a.n;
        x[2] = (D == 2) ? 0 : rr / a.n;
        int vid = 0, mul = 1;
        bool inside = true;
#pragma unroll
        for (int k = 0; k < D; ++k) {
          const int v = x[k] + ((corner >> k) & 1);
          inside = inside && v > 0 && v < a.n;
          vid += (v - 1) * mul;
          mul *= nv;
        }
        sW[c2 * Sh::NV + corner] = inside ? cs[vid] : C(0);
      }
    }
    __syncthreads();
    const cptr<C> E = as_const(a.ref) + RefOff<N>::E;
    if constexpr (D == 3) {
      // x: [c'][b'][a'] -> sNB[cl][c'][b'][a] (a + N (b' + NC c'))
      for (int i = tid; i < nc * ncr * ncr; i += Sh::NT) {
        const int c2 = i / (ncr * ncr), rem = i % (ncr * ncr);
        C x[NCB];
#pragma unroll
        for (int j = 0; j < NCB; ++j) x[j] = j >= ncr ? C(0) : sW[c2 * Sh::NV + ncr * rem + min(j, ncr - 1)];
#pragma unroll
        for (int ax = 0; ax < N; ++ax) {
          C s = 0;
#pragma unroll
          for (int j = 0; j < NCB; ++j) s += E[ax * ncr + min(j, ncr - 1)] * x[j];  // x[j] = 0 past ncr
          sNB[c2 * Sh::NF * 2 * L + N * rem + ax] = s;
        }
      }
      __syncthreads();
      // y: sNB[c'][b'][a] -> sW[cl][c'][b][a] (a + N b + N^2 c')
      for (int i = tid; i < nc * ncr * N; i += Sh::NT) {
        const int c2 = i / (ncr * N), rem = i % (ncr * N);
        const int ax = rem % N, cz = rem / N;
        C x[NCB];
#pragma unroll
        for (int j = 0; j < NCB; ++j)
          x[j] = j >= ncr ? C(0) : sNB[c2 * Sh::NF * 2 * L + ax + N * (min(j, ncr - 1) + ncr * cz)];
#pragma unroll
        for (int by = 0; by < N; ++by) {
          C s = 0;
#pragma unroll
          for (int j = 0; j < NCB; ++j) s += E[by * ncr + min(j, ncr - 1)] * x[j];  // x[j] = 0 past ncr
          sW[c2 * Sh::NV + ax + N * by + N * N * cz] = s;
        }
      }
    } else {
      // y: [b'][a'] -> sNB[cl][b][a'] (a' + NC b)
      for (int i = tid; i < nc * ncr; i += Sh::NT) {
        const int c2 = i / ncr, ac = i % ncr;
        C x[NCB];
#pragma unroll
        for (int j = 0; j < NCB; ++j) x[j] = j >= ncr ? C(0) : sW[c2 * Sh::NV + ac + ncr * min(j, ncr - 1)];
#pragma unroll
        for (int by = 0; by < N; ++by) {
          C s = 0;
#pragma unroll
          for (int j = 0; j < NCB; ++j) s += E[by * ncr + min(j, ncr - 1)] * x[j];  // x[j] = 0 past ncr
          sNB[c2 * Sh::NF * 2 * L + ac + ncr * by] = s;
        }
      }
    }
    __syncthreads();
  }
  // the thread's own line: add the prolongated correction, store u and the
  // traces of that axis, stage u for the others
  T* trout = a.tr_out + rt;
  if (act) {
    if constexpr (NC != 0) {
      const cptr<C> E = as_const(a.ref) + RefOff<N>::E;
      const C* src = D == 3 ? sW + cl * Sh::NV + ln : sNB + cl * Sh::NF * 2 * L + ncr * ln;
      C x[NCB];
#pragma unroll
      for (int j = 0; j < NCB; ++j) x[j] = j >= ncr ? C(0) : src[min(j, ncr - 1) * ST];
#pragma unroll
      for (int az = 0; az < N; ++az) {
        C s = 0;
#pragma unroll
        for (int j = 0; j < NCB; ++j) s += E[az * ncr + min(j, ncr - 1)] * x[j];  // x[j] = 0 past ncr
        u[az] += s;
      }
#pragma unroll
      for (int j = 0; j < N; ++j) a.u_out[own + j * ST] = u[j];
    }
#pragma unroll
    for (int j = 0; j < N; ++j) sU[lds_line<D, N>(cl, F, ln) + j * lds_stride<D, N>(F)] = u[j];
    store_line_traces<T, D, N, IVAR>(a, trout, B, cl, c, mask, F, ln, u);
  }
  cell_sync<D, N>();
  if (act) store_other_traces<T, D, N, F, IVAR>(a, trout, sU, B, cl, c, mask, ln);
}

template <typename T, int D, int N, int NC, bool IVAR, bool AD = false>
__global__ __launch_bounds__((DGShape<D, N>::BLOCK)) void k_prolong(DGArgs<T> a) {
  __shared__ __attribute__((aligned(16))) char lds[prolong_lds_bytes<T, D, N, NC>()];
  int id, rhs;
  block_of_grid<D, N, AD>(a, id, rhs);
  prolong_body<T, D, N, NC, IVAR, AD>(a, id, rhs, lds);
}


// ---------------------------------------------------------------- launchers
// Kinds of traversal that this shape serves (HPMG_TILE): constant kappa,
// variable kappa, adaptive meshes.
template <typename T, int D>
constexpr bool serves_const() {
  return D == 2 || HPMG_TILE == 0 || HPMG_TILE == 3;
}
template <typename T, int D>
constexpr bool serves_vark() {
  return D == 2 || HPMG_TILE == 2 || (HPMG_TILE == 3 && sizeof(T) == 2);
}
template <typename T, int D>
constexpr bool serves_adapt() {
  return sizeof(T) >= 4 && (D == 2 || HPMG_TILE == 3);
}

// One block per brick (x layers times right-hand sides, y, z) or run of cells
// (blocks, right-hand sides); see block_of_grid.
template <int D, int N, typename T>
dim3 block_grid(const DGArgs<T>& a, int nrhs) {
  using Sh = DGShape<D, N>;
  if (Cells<D, N, false>::BR)
    return dim3(brick_layers(a.n, Sh::BX) * nrhs, brick_layers(a.n, Sh::BY), brick_layers(a.n, Sh::BZ));
  return dim3((a.ncell + Sh::CPB - 1) / Sh::CPB, nrhs);
}

template <typename C, int D, int N>
bool launch_build_eig(const DGArgs<C>& a, hipStream_t s) {
  if constexpr (serves_vark<C, D>()) {
    hipLaunchKernelGGL((k_build_eig<C, D, N>), (block_grid<D, N>(a, 1)), dim3(DGShape<D, N>::THREADS), 0, s, a);
    return true;
  }
  return false;
}

template <typename T, int D, int N, bool UZERO, bool VARK, bool IVAR, bool MF = false, bool AD = false>
void start_sweep(const DGArgs<T>& a, dim3 grid, dim3 blk, hipStream_t s) {
  if constexpr (!UZERO && sizeof(T) >= 4 && !dual_sweep<T, D, N, VARK>()) {
    if (a.gl) {
      hipLaunchKernelGGL((k_sweep<T, D, N, UZERO, VARK, IVAR, MF, AD, true>), grid, blk, 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((k_sweep<T, D, N, UZERO, VARK, IVAR, MF, AD>), grid, blk, 0, s, a);
}
template <typename T, int D, int N, int NC, bool RESID, bool VARK, bool IVAR, bool AD = false>
void start_apply(const DGArgs<T>& a, dim3 grid, dim3 blk, hipStream_t s) {
  if constexpr (!dual_apply<T, D, N, VARK>()) {
    if (a.gl) {
      hipLaunchKernelGGL((k_apply<T, D, N, NC, RESID, VARK, IVAR, AD, true>), grid, blk, 0, s, a);
      return;
    }
  }
  hipLaunchKernelGGL((k_apply<T, D, N, NC, RESID, VARK, IVAR, AD>), grid, blk, 0, s, a);
}

template <typename T, int D, int N, bool UZERO>
bool launch_sweep_u(const DGArgs<T>& a, int nrhs, hipStream_t s) {
  using Sh = DGShape<D, N>;
  const dim3 grid = block_grid<D, N>(a, nrhs);
  // matrix cores (16-bit storage, 3D): whole waves per block
  constexpr bool MF = sizeof(T) == 2 && D == 3;
  const dim3 blk(MF && a.mfma ? Sh::BLOCK : Sh::THREADS);
  if (a.adapt) {
    if constexpr (serves_adapt<T, D>()) {
      start_sweep<T, D, N, UZERO, false, false, false, true>(a, grid, blk, s);
      return true;
    }
  } else if (a.vark) {
    if constexpr (serves_vark<T, D>()) {
      if (MF && a.mfma)
        start_sweep<T, D, N, UZERO, true, false, MF>(a, grid, blk, s);
      else
        start_sweep<T, D, N, UZERO, true, false>(a, grid, blk, s);
      return true;
    }
  } else if constexpr (serves_const<T, D>()) {
    if (MF && a.mfma && a.ivar)
      start_sweep<T, D, N, UZERO, false, true, MF>(a, grid, blk, s);
    else if (MF && a.mfma)
      start_sweep<T, D, N, UZERO, false, false, MF>(a, grid, blk, s);
    else if (a.ivar)
      start_sweep<T, D, N, UZERO, false, true>(a, grid, blk, s);
    else
      start_sweep<T, D, N, UZERO, false, false>(a, grid, blk, s);
    return true;
  }
  return false;
}
template <typename T, int D, int N>
bool launch_sweep(const DGArgs<T>& a, int nrhs, bool uzero, hipStream_t s) {
  return uzero ? launch_sweep_u<T, D, N, true>(a, nrhs, s) : launch_sweep_u<T, D, N, false>(a, nrhs, s);
}

template <typename T, int D, int N, int NC, bool RESID>
bool launch_apply_r(const DGArgs<T>& a, int nrhs, hipStream_t s) {
  const dim3 grid = block_grid<D, N>(a, nrhs), blk(DGShape<D, N>::THREADS);
  if (a.adapt) {
    if constexpr (serves_adapt<T, D>()) {
      start_apply<T, D, N, NC, RESID, false, false, true>(a, grid, blk, s);
      return true;
    }
  } else if (a.vark) {
    if constexpr (serves_vark<T, D>()) {
      start_apply<T, D, N, NC, RESID, true, false>(a, grid, blk, s);
      return true;
    }
  } else if constexpr (serves_const<T, D>()) {
    if (a.ivar)
      start_apply<T, D, N, NC, RESID, false, true>(a, grid, blk, s);
    else
      start_apply<T, D, N, NC, RESID, false, false>(a, grid, blk, s);
    return true;
  }
  return false;
}
template <typename T, int D, int N, int NC>
bool launch_apply(const DGArgs<T>& a, int nrhs, bool resid, hipStream_t s) {
  return resid ? launch_apply_r<T, D, N, NC, true>(a, nrhs, s) : launch_apply_r<T, D, N, NC, false>(a, nrhs, s);
}

template <typename T, int D, int N, int NC>
bool launch_prolong(const DGArgs<T>& a, int nrhs, hipStream_t s) {
  const dim3 grid = block_grid<D, N>(a, nrhs), blk(DGShape<D, N>::THREADS);
  if (a.adapt) {
    if constexpr (serves_adapt<T, D>()) {
      hipLaunchKernelGGL((k_prolong<T, D, N, NC, false, true>), grid, blk, 0, s, a);
      return true;
    }
  } else if constexpr (serves_const<T, D>() || serves_vark<T, D>()) {
    if (a.ivar)
      hipLaunchKernelGGL((k_prolong<T, D, N, NC, true>), grid, blk, 0, s, a);
    else
      hipLaunchKernelGGL((k_prolong<T, D, N, NC, false>), grid, blk, 0, s, a);
    return true;
  }
  return false;
}

}  // namespace HPMG_DGK
}  // namespace hpmg
