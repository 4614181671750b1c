// Matrix-free SIPG kernels on DG levels (gfx950).
//
// One thread per 1D line of a cell ("pencil"): a cell of N^d nodes owns
// N^(d-1) threads; a block holds CPB whole cells (up to 512 threads), a run of
// cells that follow one another in memory or a brick of them (brick()).  The
// threads load and store lines of their cells so that a wave's accesses are
// consecutive, and apply sum-factorised 1D contractions along x, y, z with the
// line in registers, exchanging lines through LDS.
//
// Operator (paper Section 2.3.1 eq. weak_form_IP with theta = -1 and the
// facet form eq. weak_form_IP_facet_spaces): in reference units the cell
// block is the Kronecker sum A_{K<-K} = h^(d-2) sum_k M x .. x L_k x .. x M,
// L_k = kappa_K Khat + facet terms of the two facets normal to axis k.  The
// neighbour coupling enters only through the traces (value g and outward
// normal derivative q = h du/dn) that each neighbour projected onto the
// shared facet (technique projection-variables); the flux variables
// w = kappa_F (q'/2 - sigma_hat g') and w' = kappa_F g'/2 (technique
// numerical-flux-outcome) are formed in registers and lifted back with the
// facet mass.  The block inverse uses the fast diagonalisation
// A_{K<-K}^{-1} = h^(2-d) (S x S x S) diag(1/(lx+ly+lz)) (S x S x S)^T with
// L_k S = M S diag(l), S^T M S = I.
//
// Sweep (technique shift-and-fuse, Algorithm BlockJacobi with loop fusion):
// each cell reads its own u, b and the neighbours' old traces, computes
//   u_new = (1-omega) u + omega A_{K<-K}^{-1} (b - A_{c<-f} w),
// which equals u + omega A_{K<-K}^{-1}(b - A u) (block-Jacobi, eq.
// block-Jacobi-IP) because A_{K<-K}^{-1} A_{K<-K} u = u, and writes u_new
// and its traces into the other trace buffer (ping-pong, so every cell of a
// sweep sees old traces: Jacobi semantics without a copy of u).
#pragma once
#include <hip/hip_runtime.h>

namespace hpmg {

// Cells of a block (of shape V).  3D uniform meshes in FP64 and FP32: a brick
// of BX x BY x BZ cells.  A traversal knows the traces of every facet inside a
// brick from the u it holds, so only the facets between bricks go through the
// trace buffers: of the 12 N^2 trace words that a cell writes and as many that
// it reads per sweep beside its 3 N^3 of u and b, a share
// 1 - (1/BX + 1/BY + 1/BZ)/3 stays on chip (0.75 at degree 1, 0.6 at degree 4).
// 2D, adaptive and small meshes (run_cells), and 16-bit storage (whose sweep is
// bound by instruction issue, not by traffic: FP16 Q5 48^3 81 us in runs, 91 us
// in bricks): runs of consecutive cells.
//   V = 0  constant kappa (and 2D)
//   V = 1  the same with about half the cells (degree 1 to 5: tile variant of the
//          batched driver's autotuner)
//   V = 2  variable kappa, whose per-cell 1D matrices share the LDS
//   V = 3  runs of cells in 3D
// Bricks are chosen so that a workgroup has 4 or 8 nearly full waves: one of 5
// waves is allocated as two waves on every SIMD (a 2 x 2 x 2 brick of degree 5,
// 288 threads, held 20 of 32 waves per CU: FP64 48^3 sweep 283 us, against 197
// us for 7 x 2 x 1).  Sweep, runs -> bricks: FP64 Q3 64^3 227 -> 146 us, Q4 48^3
// 168 -> 121 us, Q5 48^3 252 -> 197 us; FP32 Q3 64^3 110 -> 74 us, Q5 48^3 138 -> 106 us.
// Degree 6, whose sweeps are dual, takes 5 cells: with 10 they take 1.04 to 1.07
// times as long on 15^3 to 28^3 cells.
constexpr int kTileVariants = 2;
struct Brick {
  int x, y, z;
};
__host__ __device__ constexpr Brick brick(int N, int V) {
  switch (N) {
    case 2: return V == 1 ? Brick{4, 4, 2} : Brick{4, 4, 4};
    case 3: return V == 1 ? Brick{3, 2, 2} : Brick{3, 3, 3};
    case 4: return V == 1 ? Brick{2, 2, 2} : Brick{4, 2, 2};
    case 5: return V == 0 ? Brick{5, 2, 2} : Brick{5, 2, 1};
    case 6: return V == 0 ? Brick{7, 2, 1} : Brick{3, 2, 1};
    case 7: return Brick{5, 1, 1};
    case 8: return Brick{2, 2, 1};
    default: return Brick{3, 1, 1};
  }
}
__host__ __device__ constexpr int cells_per_block_v(int D, int N, int V) {
  if (D == 2) return 256 / N;
  if (V == 3) return 256 / (N * N);
  return brick(N, V).x * brick(N, V).y * brick(N, V).z;
}
// Blocks of a 3D uniform mesh with n cells per axis, and the facet records
// (2 N^2 values each) that one trace buffer holds: for every axis the lower
// and upper faces of the bricks, n^2 facets per layer of bricks.
__host__ __device__ constexpr int brick_layers(int n, int b) { return (n + b - 1) / b; }
inline long long brick_blocks(int n, int N, int V) {
  const Brick b = brick(N, V);
  return (long long)brick_layers(n, b.x) * brick_layers(n, b.y) * brick_layers(n, b.z);
}
inline long long brick_records(int n, int N, int V) {
  const Brick b = brick(N, V);
  return 2LL * n * n * (brick_layers(n, b.x) + brick_layers(n, b.y) + brick_layers(n, b.z));
}
// Shape of the blocks of a 3D uniform mesh with constant kappa in FP64 or FP32,
// the same for every operation on a level: runs of cells (V = 3) on meshes of at
// most so many full bricks' cells, bricks (V = 0) above.  Small meshes leave
// bricks, larger blocks than runs with a step more, few to a chip of 256 CUs, and
// their ragged ones half empty: four sweeps in bricks | runs, FP64 degree 4, 8^3
// cells 39 | 30 us, degree 6, 6^3 61 | 41, degree 1, 24^3 22.7 | 24.1; FP32 degree 1,
// 16^3 26.7 | 24.4.  In FP32 the dual form (dual_sweep, dual_apply) gains so little
// from bricks, whose passes it has beside one step more, that degree 4, 5 and 8
// stay in runs up to 28^3, 30^3 and 13^3 cells (degree 5, 22^3, sweeps 72 | 62 us,
// apply 24 | 20.5) and degree 6 always (27^3, sweeps 176 | 149).
__host__ __device__ constexpr int run_cells(int N, bool fp64) {
  constexpr int line[2][8] = {{400, 400, 160, 1400, 2000, 1 << 24, 160, 800}, {200, 200, 160, 160, 1000, 300, 160, 200}};
  const long long c = (long long)line[fp64 ? 1 : 0][N - 2] * cells_per_block_v(3, N, 0);
  return c < (1 << 30) ? (int)c : 1 << 30;
}
__host__ __device__ constexpr int mesh_variant(int n, int N, bool fp64) {
  return (long long)n * n * n <= run_cells(N, fp64) ? 3 : 0;
}
// Block index of a brick (10 bits per axis; a 3D mesh has n <= 1023).
__host__ __device__ constexpr int brick_id(int x, int y, int z) { return x | (y << 10) | (z << 20); }
template <int D, int N, int V>
struct DGShapeV {
  static constexpr int L = (D == 2) ? N : N * N;  // lines per cell = nodes per facet
  static constexpr int NV = L * N;                // nodes per cell
  static constexpr int NF = 2 * D;                // facets per cell
  // LDS row of a cell along x, padded for N = 4 and 8 so that the lines of a
  // wave along every axis fall into different banks (N = 8 in FP32: 8 lanes per
  // bank without it; FP64 apply 32^3 169 -> 143 us, FP32 90 -> 71 us; N = 4,
  // 64^3, 165 -> 147 and 90 -> 74 us; N = 6, two lanes per bank, 2% slower with
  // it), and nodes of a cell with the padding
  static constexpr int SY = N + (N % 4 == 0 ? 1 : 0), NVP = (D == 2 ? 1 : N) * N * SY;
  static constexpr int BX = brick(N, V).x, BY = brick(N, V).y, BZ = brick(N, V).z;  // 3D
  static constexpr int CPB = cells_per_block_v(D, N, V);
  static constexpr int NT = CPB * L;
  // 3D cells whose L lines fill (nearly) whole waves, CPW cells in each (degree
  // 1, 2, 3 and 7: 16, 7, 4 and 1): no cell is split between waves, so the
  // steps of a traversal that exchange lines within a cell need no barrier
  // (cell_sync)
  static constexpr int CPW = (D == 3 && L <= 64) ? 64 / L : 1;
  static constexpr bool WAVE = D == 3 && L <= 64 && 64 - CPW * L <= 1;
  static constexpr int BLOCK = WAVE ? (CPB + CPW - 1) / CPW * 64 : (NT + 63) / 64 * 64;  // whole waves
  static constexpr int THREADS = WAVE ? BLOCK : NT;  // launched
  static constexpr int EGS = 2 * N * N + N;       // S, Si, lambda of one direction (class tables)
  static constexpr int EGV = N * N + N;           // S, lambda of one direction (per cell, variable kappa)
};
template <int D, int N>
using DGShape = DGShapeV<D, N, 0>;

// Per-level reference data (type T), in global memory:
//   [0, N^2)            Mhat (1D mass on [0,1], symmetric)
//   [N^2, N^2+N)        ep0: outward normal derivative functional at x=0
//   [N^2+N, N^2+2N)     ep1: same at x=1
//   [N^2+2N, N^2+3N)    ev0: value functional at x=0 (used with gl)
//   [N^2+3N, N^2+4N)    ev1: value functional at x=1
//   [N^2+4N, N^2+5N)    al0: lift of a neighbour's normal derivative q' across
//                       the facet at x=0, nodal (see nodal_lifts); mirrored at x=1
//   [N^2+5N, N^2+6N)    be0: the same of its value g'
//   then four compact even-odd tables (EO<N>::SIZE each): Mhat, Mhat^-1, and
//   for constant kappa S and Si^T of the interior class
//   [E, ...)            interpolation to the fine nodes from the next
//                       coarser nodes, E[a*NC + j] (only when NC > 0)
template <int N>
struct RefOff {
  static constexpr int Q = ((N + 1) / 2) * ((N + 1) / 2) + (N / 2) * (N / 2);
  static constexpr int M = 0, EP0 = N * N, EP1 = N * N + N, EV0 = N * N + 2 * N, EV1 = N * N + 3 * N,
                       AL0 = N * N + 4 * N, BE0 = N * N + 5 * N, MC = N * N + 6 * N, MIC = MC + Q, SC = MC + 2 * Q,
                       SIC = MC + 3 * Q, E = MC + 4 * Q;
};

// Storage type T of the cell vectors and traces, compute type CT<T> of the
// arithmetic, LDS, operator tables and coarse-level vectors: half-precision
// storage (FP16 or BF16) computes in FP32.
template <typename T>
struct Compute {
  using type = T;
};
template <>
struct Compute<_Float16> {
  using type = float;
};
template <>
struct Compute<__bf16> {
  using type = float;
};
template <typename T>
using CT = typename Compute<T>::type;

template <typename T>
struct DGArgs {
  using C = CT<T>;
  int n, ncell;
  int vark;            // 0: class tables (constant kappa), 1: per-cell eigendata + kappa
  int gl;              // 0: Gauss-Lobatto nodes (facet values are the end nodes), 1: Gauss-Legendre
  C kappa_const;
  const C* ref;        // RefOff layout
  const C* eig;        // vark=0: [4 classes][S N^2 | Si N^2 | lam N]; vark=1: [cell][D][S N^2 | lam N]
  const C* kappa;      // vark=1: per cell
  const C* rk;         // vark=1 with the block recomputed in each traversal: [Khat | C^-1] (Mhat = C C^T),
                       // eig unused; nullptr: eig holds the precomputed per-cell data
  const unsigned char* bmask;  // per cell: bit 2k+side set if that facet is on the boundary
  C h_fwd;             // h^(2-d): scales b in the sweep
  C h_apply;           // h^(d-2): scales A u
  C sigma_hat;         // sigma * h = sigma0 (p_penalty+1)^2
  C omega;
  const T* u_in;       // cell vector
  T* u_out;            // cell vector (may alias u_in)
  const T* b;          // cell vector
  const T* tr_in;      // traces, records of L pairs (value, derivative): 2D and adaptive meshes [2D][ncell] (then
                       // the hanging-facet slots), 3D the faces of the bricks (Cells::own_rec)
  T* tr_out;
  C* out;              // apply: y; resid: r (NC=0) or coarse right-hand side (next level, compute type)
  const C* coarse;     // prolong: coarse cell vector (DG) or Q1 interior vertex vector (CG)
  int coarse_cg;       // prolong partner: 0 DG, 1 Q1 (vertex gather), 2 Q1 corner values per cell [c][2^d]
  long long vstride;   // per right-hand side stride of cell vectors
  long long tstride;   // per right-hand side stride of trace buffers
  long long cstride;   // per right-hand side stride of coarse vectors
  // Fusions of the outer FP64 Krylov iteration into the finest-level
  // kernels (one right-hand side, NC = 0, T = double):
  //   kry = 1 (projection): first p = z + beta p in place (u_in = u_out = p),
  //     z of type zkind (hpmg_dtype code) at zlow, read as
  //     z * (zscaled ? kscal[8] / kmul : 1), beta = kscal[3]
  //   kdot = 1 (apply, y = A p): kpartial[block] = the block's share of p.y
  int kry = 0, kdot = 0, zkind = 0, zscaled = 0;
  // Interior-block smoother (constant kappa; Section 4.1 technique
  // approximate boundary operators): ivar = 1 takes the block of an interior
  // cell (class 0 along every axis) as the block-Jacobi block D~ of every
  // cell.  The operator stays A: a boundary facet contributes the lift of
  // the cell's own traces with the sign reversed, i.e. (D~ - A_{K<-K}) u
  // (the difference of the two 1D operators is the boundary-facet term,
  // kappa/2 (e ep^T + ep e^T) - sigma_hat kappa e e^T), so that the sweep
  // computes u + omega D~^-1 (b - A u) and the apply A u.  In 2D traces are
  // then stored on boundary facets too.
  int ivar = 0;
  // Variable kappa in 3D, FP64, sweeps with u != 0 on entry: the right-hand
  // side in nodal form, h_fwd b times Mhat^-1 along every axis, as
  // [cell][node of the x line][line]; bp_mode 1 stores it, 2 reads it instead
  // of forming it from b; vstride per right-hand side.
  C* bp = nullptr;
  int bp_mode = 0;
  int ncd = 0;         // nodes per direction of the coarse DG level (transfers with a run-time degree)
  // 16-bit storage sweeps (3D): 1 runs the six volume contractions of the
  // block solve on the matrix cores (16-bit operands, FP32 accumulation);
  // 0 keeps them on the vector units in FP32
  int mfma = 0;
  // Adaptive (spacetree) meshes with constant kappa (Section 2.1; the
  // kernels' AD instances): amask[c] holds bit f if facet f of cell c lies
  // on the boundary and bit 8 + f if facet f is the coarse side of a
  // hanging facet (r^(d-1) finer neighbours, penalty sig_hang = r
  // sigma_hat); nbslot[f ncell + c] is the trace slot (unit 2L values)
  // that holds the neighbour-side traces of facet f in the neighbour's
  // reference units: the neighbour's own slot (f^1) ncell + c' across a
  // conforming facet, else a slot filled by the hanging-facet remap;
  // hscale[c] = (h_base / h_c)^(d-2) (nullptr: 1); mort = the remap
  // tables of the level (host side only).
  int adapt = 0;
  C sig_hang = 0;
  const unsigned short* amask = nullptr;
  const int* nbslot = nullptr;
  const C* hscale = nullptr;
  const C* mort = nullptr;
  const int* itab = nullptr;   // hanging interfaces (host side: the remap launch)
  int nif = 0, mif = 0, rfac = 0;
  int* flag = nullptr;  // eigendata build: set to 1 if a block eigenvalue is not positive and finite
  const void* zlow = nullptr;
  const double* kscal = nullptr;
  double kmul = 1.0;
  double* kpartial = nullptr;
};

}  // namespace hpmg
