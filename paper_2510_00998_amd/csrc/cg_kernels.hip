// Kernels of the continuous Q1 levels (paper Section 2.4 point-Jacobi with
// the accumulated diagonal; Section 5.2 h-multigrid), the DG -> Q1 gather of
// restricted residuals, the dense coarsest solve, and the FP64 vector
// operations of the outer Krylov iteration.
#include <hip/hip_runtime.h>

#include "cg_block.hpp"
#include "cg_tiles.hpp"
#include "kernels.hpp"

namespace hpmg {

namespace {

template <int D>
__device__ __forceinline__ void vcoords(int v, int nv, int (&x)[3]) {
  x[0] = v % nv;
  x[1] = (v / nv) % nv;
  x[2] = (D == 3) ? v / (nv * nv) : 0;
}

// out = u + omega Dinv (b - A u)   (mode 0; u = 0 if uzero)
// out = b - A u                    (mode 1)
// at vertex v (total = nv^d).  The stencil is stored point-major,
// st[s * nv^d + v], so that a wave reads each stencil point of its vertices
// with one coalesced load.  Neighbour indices are clamped into the grid
// instead of skipped: the stencil entry of a neighbour outside the interior
// is zero, and the loads of a thread are independent of each other.
template <typename T, int D>
__device__ __forceinline__ T cg_stencil_at(int v, int nv, int total, const T* __restrict__ st,
                                           const T* __restrict__ dinv, const T* __restrict__ u,
                                           const T* __restrict__ b, T omega, int mode, int uzero) {
  constexpr int NS = (D == 2) ? 9 : 27;
  T au = 0;
  if (!uzero) {
    int x[3];
    vcoords<D>(v, nv, x);
    int cx[3], cy[3], cz[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      cx[d] = min(max(x[0] + d - 1, 0), nv - 1);
      cy[d] = min(max(x[1] + d - 1, 0), nv - 1) * nv;
      cz[d] = (D == 3) ? min(max(x[2] + d - 1, 0), nv - 1) * nv * nv : 0;
    }
    T sv[NS], uv[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      sv[s] = st[(size_t)s * total + v];
      uv[s] = u[cx[s % 3] + cy[(s / 3) % 3] + cz[(D == 3) ? s / 9 : 1]];
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) au += sv[s] * uv[s];
  }
  if (mode == 0) {
    const T u0 = uzero ? T(0) : u[v];
    return u0 + omega * dinv[v] * (b[v] - au);
  }
  return b[v] - au;
}

template <typename T, int D>
__global__ __launch_bounds__(256) void k_cg_stencil(int nv, const T* __restrict__ st, const T* __restrict__ dinv,
                                                    const T* __restrict__ u, const T* __restrict__ b,
                                                    T* __restrict__ out, T omega, int mode, int uzero) {
  const int total = (D == 2) ? nv * nv : nv * nv * nv;
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= total) return;
  out[v] = cg_stencil_at<T, D>(v, nv, total, st, dinv, u, b, omega, mode, uzero);
}

template <typename T, int D, int RK>
__global__ __launch_bounds__(256) void k_cg_restrict(int nvf, int nvc, const int* __restrict__ ridx,
                                                     const T* __restrict__ rw, const T* __restrict__ rf,
                                                     T* __restrict__ bc) {
  const int total = (D == 2) ? nvc * nvc : nvc * nvc * nvc;
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= total) return;
  int x[3];
  vcoords<D>(v, nvc, x);
  bc[v] = cgt::restrict_box<T, D, RK>(cgt::Parents<T, D, RK>(ridx, rw, x, {0, 0, 0}), {0, 0, 0}, nvf, rf);
}

// u_f += P e_c
template <typename T, int D>
__global__ __launch_bounds__(256) void k_cg_prolong(int nvf, int nvc, const int* __restrict__ pidx,
                                                    const T* __restrict__ pw, const T* __restrict__ ec,
                                                    T* __restrict__ uf) {
  const int total = (D == 2) ? nvf * nvf : nvf * nvf * nvf;
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= total) return;
  int x[3];
  vcoords<D>(v, nvf, x);
  uf[v] += cgt::prolong_xyz<T, D>(cgt::Parents<T, D, 2>(pidx, pw, x, {0, 0, 0}), nvc, ec);
}

// Q1 right-hand side from the per-cell corner contributions of the
// restricted DG residual: b_V = sum over the 2^d cells around V.
template <typename T, int D>
__global__ __launch_bounds__(256) void k_gather_corners(int n, const T* __restrict__ contrib, T* __restrict__ bcg) {
  const int nv = n - 1;
  const int total = (D == 2) ? nv * nv : nv * nv * nv;
  const int v = blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= total) return;
  int x[3];
  vcoords<D>(v, nv, x);
  bcg[v] = cgt::gather_corners_at<T, D>(x, n, contrib);
}

// (Ainv b)_i on the coarsest level (dense FP64 inverse from a Cholesky
// factorisation done at setup), four independent loads in flight.
template <typename T>
__device__ __forceinline__ T dense_at(int i, int m, const double* __restrict__ Ainv, const T* __restrict__ b) {
  const double* row = Ainv + (size_t)i * m;
  double s = 0.0;
  int j = 0;
  for (; j + 4 <= m; j += 4) {
    const double a0 = row[j], a1 = row[j + 1], a2 = row[j + 2], a3 = row[j + 3];
    const double b0 = (double)b[j], b1 = (double)b[j + 1], b2 = (double)b[j + 2], b3 = (double)b[j + 3];
    s += a0 * b0;
    s += a1 * b1;
    s += a2 * b2;
    s += a3 * b3;
  }
  for (; j < m; ++j) s += row[j] * (double)b[j];
  return (T)s;
}

template <typename T>
__global__ __launch_bounds__(256) void k_dense_solve(int m, const double* __restrict__ Ainv, const T* __restrict__ b,
                                                     T* __restrict__ x) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  x[i] = dense_at<T>(i, m, Ainv, b);
}

// Coarse vertices per axis and tile.
template <int D, int RK>
constexpr int tile_ct() {
  return D == 3 ? 2 : (RK == 3 ? 8 : 4);
}
template <typename T, int D, int RK, int NU>
__global__ __launch_bounds__((cgt::Tile<D, RK, tile_ct<D, RK>()>::THREADS)) void k_cg_down(CGTileArgs<T> a) {
  __shared__ __attribute__((aligned(16))) char lds[cgt::Tile<D, RK, tile_ct<D, RK>()>::template lds_bytes<T>()];
  cgt::down_tile<T, D, RK, tile_ct<D, RK>(), NU>(a, blockIdx.x, blockIdx.y, lds);
}
template <typename T, int D, int RK, int NU>
__global__ __launch_bounds__((cgt::Tile<D, RK, tile_ct<D, RK>()>::THREADS)) void k_cg_up(CGTileArgs<T> a) {
  __shared__ __attribute__((aligned(16))) char lds[cgt::Tile<D, RK, tile_ct<D, RK>()>::template lds_bytes<T>()];
  cgt::up_tile<T, D, RK, tile_ct<D, RK>(), NU>(a, blockIdx.x, blockIdx.y, lds);
}

template <typename T, int D, int RK>
__global__ __launch_bounds__(CG_BLOCK_MAX_VERTICES) void k_cg_vcycle_block(CGBlockArgs<T> a) {
  __shared__ cgb::Lds<T> lds;
  cgb::vcycle<T, D, RK>(a, blockIdx.x, lds);
}

template <typename T>
__global__ __launch_bounds__(256) void k_fill(T* __restrict__ x, size_t n, T v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) x[i] = v;
}

// ------------------------------------------------------------- FP64 Krylov
constexpr int RED_BLOCKS = 1024;

__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) s += sh[i];
  return s;
}

// partial[k*RED_BLOCKS + blk] for up to two dot products
__global__ __launch_bounds__(256) void k_dot2(size_t n, const double* __restrict__ x, const double* __restrict__ y,
                                              const double* __restrict__ z, double* __restrict__ partial) {
  __shared__ double sh[4];
  double s0 = 0.0, s1 = 0.0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const double xi = x[i];
    s0 += xi * y[i];
    if (z) s1 += xi * z[i];
  }
  double t0 = block_sum(s0, sh);
  __syncthreads();
  double t1 = block_sum(s1, sh);
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = t0;
    partial[RED_BLOCKS + blockIdx.x] = t1;
  }
}

// Low-precision z of a mixed cycle, read as z_i = (double) zl_i * sc.
template <typename T>
__device__ __forceinline__ double lowz(const T* __restrict__ zl, size_t i, double sc) {
  return (double)(float)zl[i] * sc;
}
__device__ __forceinline__ double lowz_scale(const double* __restrict__ s, int scaled, double mul) {
  return scaled ? s[8] / mul : 1.0;
}

// partials of z.r and z.rold with z read from the cycle's own vector (no
// FP64 copy of z is formed)
template <typename T>
__global__ __launch_bounds__(256) void k_dot2z(size_t n, const T* __restrict__ zl, const double* __restrict__ s,
                                               int scaled, double mul, const double* __restrict__ r,
                                               const double* __restrict__ rold, double* __restrict__ partial) {
  __shared__ double sh[4];
  const double sc = lowz_scale(s, scaled, mul);
  double s0 = 0.0, s1 = 0.0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const double zi = lowz(zl, i, sc);
    s0 += zi * r[i];
    s1 += zi * rold[i];
  }
  double t0 = block_sum(s0, sh);
  __syncthreads();
  double t1 = block_sum(s1, sh);
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = t0;
    partial[RED_BLOCKS + blockIdx.x] = t1;
  }
}

// Sum the partials into slots and apply the scalar step of the flexible CG:
//  op 0: s[a0] = sum0
//  op 1: beta: s[3] = first ? 0 : (sum0 - sum1)/s[2]; s[2] = sum0 (rho)
//  op 2: alpha: s[5] = s[2] / sum0
//  op 3: s[6] = sum0 (r.r), s[7] = 1/sqrt(sum0), s[8] = sqrt(sum0)
__global__ __launch_bounds__(256) void k_finalize(const double* __restrict__ partial, int nblk, double* __restrict__ s,
                                                  int op, int a0, int first) {
  __shared__ double sh[4];
  double v0 = 0.0, v1 = 0.0;
  for (int i = threadIdx.x; i < nblk; i += blockDim.x) {
    v0 += partial[i];
    v1 += partial[RED_BLOCKS + i];
  }
  const double t0 = block_sum(v0, sh);
  __syncthreads();
  const double t1 = block_sum(v1, sh);
  if (threadIdx.x == 0) {
    if (op == 0) {
      s[a0] = t0;
    } else if (op == 1) {
      s[3] = first ? 0.0 : (t0 - t1) / s[2];
      s[2] = t0;
    } else if (op == 2) {
      s[5] = s[2] / t0;
    } else {
      s[6] = t0;
      s[7] = t0 > 0.0 ? 1.0 / sqrt(t0) : 1.0;
      s[8] = sqrt(t0);
    }
  }
}

// alpha = rho / p.q from the per-block shares of p.q: s[5] = s[2] / sum
__global__ __launch_bounds__(256) void k_finalize_alpha(const double* __restrict__ partial, int n,
                                                        double* __restrict__ s) {
  __shared__ double sh[4];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) v += partial[i];
  const double t = block_sum(v, sh);
  if (threadIdx.x == 0) s[5] = s[2] / t;
}

// y += a x
__global__ __launch_bounds__(256) void k_axpy(size_t n, double a, const double* __restrict__ x, double* __restrict__ y) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    y[i] += a * x[i];
}

// p = z + beta p (p = z when beta == 0: the first iteration never reads
// the previous search direction)
__global__ __launch_bounds__(256) void k_update_p(size_t n, const double* __restrict__ z, double* __restrict__ p,
                                                  const double* __restrict__ s) {
  const double beta = s[3];
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = beta == 0.0 ? z[i] : z[i] + beta * p[i];
}

// p = z + beta p with z read from the cycle's low-precision vector
template <typename T>
__global__ __launch_bounds__(256) void k_update_pz(size_t n, const T* __restrict__ zl, double* __restrict__ p,
                                                   const double* __restrict__ s, int scaled, double mul) {
  const double beta = s[3];
  const double sc = lowz_scale(s, scaled, mul);
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const double zi = lowz(zl, i, sc);
    p[i] = beta == 0.0 ? zi : zi + beta * p[i];
  }
}

// u += alpha p; r_old = r; r -= alpha q; partial r.r; r32 = (float) r when
// given (the unscaled FP32 copy that the next FP32 cycle reads)
__global__ __launch_bounds__(256) void k_update_ur(size_t n, double* __restrict__ u, double* __restrict__ r,
                                                   double* __restrict__ rold, const double* __restrict__ p,
                                                   const double* __restrict__ q, const double* __restrict__ s,
                                                   double* __restrict__ partial, float* __restrict__ r32) {
  __shared__ double sh[4];
  const double alpha = s[5];
  double acc = 0.0;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    u[i] += alpha * p[i];
    const double ri = r[i];
    rold[i] = ri;
    const double rn = ri - alpha * q[i];
    r[i] = rn;
    if (r32) r32[i] = (float)rn;
    acc += rn * rn;
  }
  const double t = block_sum(acc, sh);
  if (threadIdx.x == 0) {
    partial[blockIdx.x] = t;
    partial[RED_BLOCKS + blockIdx.x] = 0.0;
  }
}

// y = (T)(x * s[7] * mul): scaled cast for a reduced-precision cycle (s[7] =
// 1/||x||; mul = 1 for FP32, sqrt(n) for 16-bit storage so that the entries
// have unit mean square); s = null: y = (T)(x * mul)
template <typename T>
__global__ __launch_bounds__(256) void k_cast_down(size_t n, const double* __restrict__ x, T* __restrict__ y,
                                                   const double* __restrict__ s, double mul) {
  const double sc = s ? s[7] * mul : mul;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    y[i] = (T)(float)(x[i] * sc);
}

// y = (double)x * s[8] / mul
template <typename T>
__global__ __launch_bounds__(256) void k_cast_up(size_t n, const T* __restrict__ x, double* __restrict__ y,
                                                 const double* __restrict__ s, double mul) {
  const double sc = s[8] / mul;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    y[i] = (double)(float)x[i] * sc;
}

inline unsigned nblocks(size_t n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }
inline unsigned gs_blocks(size_t n) {
  size_t b = (n + 255) / 256;
  return (unsigned)(b < RED_BLOCKS ? (b ? b : 1) : RED_BLOCKS);
}

}  // namespace

template <typename T>
void cg_stencil(int D, int nv, const T* st, const T* dinv, const T* u, const T* b, T* out, T omega, int mode,
                int uzero, hipStream_t s) {
  const size_t total = (D == 2) ? (size_t)nv * nv : (size_t)nv * nv * nv;
  if (D == 2)
    hipLaunchKernelGGL((k_cg_stencil<T, 2>), dim3(nblocks(total)), dim3(256), 0, s, nv, st, dinv, u, b, out, omega, mode,
                       uzero);
  else
    hipLaunchKernelGGL((k_cg_stencil<T, 3>), dim3(nblocks(total)), dim3(256), 0, s, nv, st, dinv, u, b, out, omega, mode,
                       uzero);
}

template <typename T>
void cg_restrict(int D, int nvf, int nvc, int rk, const int* ridx, const T* rw, const T* rf, T* bc, hipStream_t s) {
  const size_t total = (D == 2) ? (size_t)nvc * nvc : (size_t)nvc * nvc * nvc;
  const dim3 g(nblocks(total));
  if (D == 2 && rk == 3)
    hipLaunchKernelGGL((k_cg_restrict<T, 2, 3>), g, dim3(256), 0, s, nvf, nvc, ridx, rw, rf, bc);
  else if (D == 2)
    hipLaunchKernelGGL((k_cg_restrict<T, 2, 5>), g, dim3(256), 0, s, nvf, nvc, ridx, rw, rf, bc);
  else if (rk == 3)
    hipLaunchKernelGGL((k_cg_restrict<T, 3, 3>), g, dim3(256), 0, s, nvf, nvc, ridx, rw, rf, bc);
  else
    hipLaunchKernelGGL((k_cg_restrict<T, 3, 5>), g, dim3(256), 0, s, nvf, nvc, ridx, rw, rf, bc);
}

template <typename T>
void cg_prolong(int D, int nvf, int nvc, const int* pidx, const T* pw, const T* ec, T* uf, hipStream_t s) {
  const size_t total = (D == 2) ? (size_t)nvf * nvf : (size_t)nvf * nvf * nvf;
  if (D == 2)
    hipLaunchKernelGGL((k_cg_prolong<T, 2>), dim3(nblocks(total)), dim3(256), 0, s, nvf, nvc, pidx, pw, ec, uf);
  else
    hipLaunchKernelGGL((k_cg_prolong<T, 3>), dim3(nblocks(total)), dim3(256), 0, s, nvf, nvc, pidx, pw, ec, uf);
}

template <typename T>
void gather_corners(int D, int n, const T* contrib, T* bcg, hipStream_t s) {
  const size_t nv = n - 1;
  const size_t total = (D == 2) ? nv * nv : nv * nv * nv;
  if (D == 2)
    hipLaunchKernelGGL((k_gather_corners<T, 2>), dim3(nblocks(total)), dim3(256), 0, s, n, contrib, bcg);
  else
    hipLaunchKernelGGL((k_gather_corners<T, 3>), dim3(nblocks(total)), dim3(256), 0, s, n, contrib, bcg);
}

template <typename T>
void dense_solve(int m, const double* Ainv, const T* b, T* x, hipStream_t s) {
  hipLaunchKernelGGL((k_dense_solve<T>), dim3(nblocks(m)), dim3(256), 0, s, m, Ainv, b, x);
}

template <typename T, int D, int RK>
void cg_tile(bool down, int nu, const CGTileArgs<T>& a, int ncol, hipStream_t s) {
  const dim3 t(cgt::Tile<D, RK, tile_ct<D, RK>()>::THREADS);
  const dim3 g(down ? cgt::down_tiles<D, tile_ct<D, RK>()>(a.nvc) : cgt::up_tiles<D, RK, tile_ct<D, RK>()>(a.nv), ncol);
  if (down && nu == 1)
    hipLaunchKernelGGL((k_cg_down<T, D, RK, 1>), g, t, 0, s, a);
  else if (down)
    hipLaunchKernelGGL((k_cg_down<T, D, RK, 2>), g, t, 0, s, a);
  else if (nu == 1)
    hipLaunchKernelGGL((k_cg_up<T, D, RK, 1>), g, t, 0, s, a);
  else
    hipLaunchKernelGGL((k_cg_up<T, D, RK, 2>), g, t, 0, s, a);
}
template <typename T>
void cg_tile_rk(bool down, int D, int rk, int nu, const CGTileArgs<T>& a, int ncol, hipStream_t s) {
  if (D == 2 && rk == 3)
    cg_tile<T, 2, 3>(down, nu, a, ncol, s);
  else if (D == 2)
    cg_tile<T, 2, 5>(down, nu, a, ncol, s);
  else if (rk == 3)
    cg_tile<T, 3, 3>(down, nu, a, ncol, s);
  else
    cg_tile<T, 3, 5>(down, nu, a, ncol, s);
}
template <typename T>
void cg_down(int D, int rk, int nu, const CGTileArgs<T>& a, int ncol, hipStream_t s) {
  cg_tile_rk<T>(true, D, rk, nu, a, ncol, s);
}
template <typename T>
void cg_up(int D, int rk, int nu, const CGTileArgs<T>& a, int ncol, hipStream_t s) {
  cg_tile_rk<T>(false, D, rk, nu, a, ncol, s);
}

template <typename T>
void cg_vcycle_block(int D, int rk, const CGBlockArgs<T>& a, int ncol, hipStream_t s) {
  const dim3 g(ncol), t(CG_BLOCK_MAX_VERTICES);
  if (D == 2 && rk == 3)
    hipLaunchKernelGGL((k_cg_vcycle_block<T, 2, 3>), g, t, 0, s, a);
  else if (D == 2)
    hipLaunchKernelGGL((k_cg_vcycle_block<T, 2, 5>), g, t, 0, s, a);
  else if (rk == 3)
    hipLaunchKernelGGL((k_cg_vcycle_block<T, 3, 3>), g, t, 0, s, a);
  else
    hipLaunchKernelGGL((k_cg_vcycle_block<T, 3, 5>), g, t, 0, s, a);
}

template <typename T>
void fill(T* x, size_t n, T v, hipStream_t s) {
  unsigned g = nblocks(n);
  if (g > 8192) g = 8192;
  if (g == 0) g = 1;
  hipLaunchKernelGGL((k_fill<T>), dim3(g), dim3(256), 0, s, x, n, v);
}

void krylov_dot(size_t n, const double* x, const double* y, const double* z, double* partial, double* scal, int op,
                int a0, int first, hipStream_t s) {
  const unsigned g = gs_blocks(n);
  hipLaunchKernelGGL(k_dot2, dim3(g), dim3(256), 0, s, n, x, y, z, partial);
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, partial, (int)g, scal, op, a0, first);
}

void krylov_alpha(const double* partial, int n, double* scal, hipStream_t s) {
  hipLaunchKernelGGL(k_finalize_alpha, dim3(1), dim3(256), 0, s, partial, n, scal);
}

void axpy(size_t n, double a, const double* x, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_axpy, dim3(gs_blocks(n)), dim3(256), 0, s, n, a, x, y);
}

void krylov_update_p(size_t n, const double* z, double* p, const double* scal, hipStream_t s) {
  hipLaunchKernelGGL(k_update_p, dim3(gs_blocks(n)), dim3(256), 0, s, n, z, p, scal);
}

void krylov_update_ur(size_t n, double* u, double* r, double* rold, const double* p, const double* q, double* partial,
                      double* scal, float* r32, hipStream_t s) {
  const unsigned g = gs_blocks(n);
  hipLaunchKernelGGL(k_update_ur, dim3(g), dim3(256), 0, s, n, u, r, rold, p, q, scal, partial, r32);
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, partial, (int)g, scal, 3, 0, 0);
}

template <typename T>
void krylov_dot_lowz(size_t n, const T* zl, int scaled, double mul, const double* r, const double* rold,
                     double* partial, double* scal, int first, hipStream_t s) {
  const unsigned g = gs_blocks(n);
  hipLaunchKernelGGL((k_dot2z<T>), dim3(g), dim3(256), 0, s, n, zl, scal, scaled, mul, r, rold, partial);
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, s, partial, (int)g, scal, 1, 0, first);
}
template <typename T>
void krylov_update_p_lowz(size_t n, const T* zl, int scaled, double mul, double* p, const double* scal,
                          hipStream_t s) {
  hipLaunchKernelGGL((k_update_pz<T>), dim3(gs_blocks(n)), dim3(256), 0, s, n, zl, p, scal, scaled, mul);
}
#define HPMG_LOWZ(T)                                                                                            \
  template void krylov_dot_lowz<T>(size_t, const T*, int, double, const double*, const double*, double*, double*, \
                                   int, hipStream_t);                                                           \
  template void krylov_update_p_lowz<T>(size_t, const T*, int, double, double*, const double*, hipStream_t);
HPMG_LOWZ(float)
HPMG_LOWZ(_Float16)
HPMG_LOWZ(__bf16)
#undef HPMG_LOWZ

template <typename T>
void cast_down(size_t n, const double* x, T* y, const double* scal, double mul, hipStream_t s) {
  hipLaunchKernelGGL((k_cast_down<T>), dim3(gs_blocks(n)), dim3(256), 0, s, n, x, y, scal, mul);
}
template <typename T>
void cast_up(size_t n, const T* x, double* y, const double* scal, double mul, hipStream_t s) {
  hipLaunchKernelGGL((k_cast_up<T>), dim3(gs_blocks(n)), dim3(256), 0, s, n, x, y, scal, mul);
}
template void cast_down<float>(size_t, const double*, float*, const double*, double, hipStream_t);
template void cast_down<_Float16>(size_t, const double*, _Float16*, const double*, double, hipStream_t);
template void cast_down<__bf16>(size_t, const double*, __bf16*, const double*, double, hipStream_t);
template void cast_up<float>(size_t, const float*, double*, const double*, double, hipStream_t);
template void cast_up<_Float16>(size_t, const _Float16*, double*, const double*, double, hipStream_t);
template void cast_up<__bf16>(size_t, const __bf16*, double*, const double*, double, hipStream_t);

#define HPMG_INST(T)                                                                                           \
  template void cg_stencil<T>(int, int, const T*, const T*, const T*, const T*, T*, T, int, int, hipStream_t); \
  template void cg_restrict<T>(int, int, int, int, const int*, const T*, const T*, T*, hipStream_t);           \
  template void cg_prolong<T>(int, int, int, const int*, const T*, const T*, T*, hipStream_t);                 \
  template void gather_corners<T>(int, int, const T*, T*, hipStream_t);                                        \
  template void dense_solve<T>(int, const double*, const T*, T*, hipStream_t);                                 \
  template void cg_down<T>(int, int, int, const CGTileArgs<T>&, int, hipStream_t);                             \
  template void cg_up<T>(int, int, int, const CGTileArgs<T>&, int, hipStream_t);                               \
  template void cg_vcycle_block<T>(int, int, const CGBlockArgs<T>&, int, hipStream_t);                         \
  template void fill<T>(T*, size_t, T, hipStream_t);
HPMG_INST(float)
HPMG_INST(double)
#undef HPMG_INST
template void fill<_Float16>(_Float16*, size_t, _Float16, hipStream_t);
template void fill<__bf16>(__bf16*, size_t, __bf16, hipStream_t);

}  // namespace hpmg
