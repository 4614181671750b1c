// Instantiation of the DG cell kernels for dim = 2, storage type double, degree
// 6 to 8, with plain 1D products in place of the even-odd ones (block_mv), for
// meshes whose blocks the chip holds at once.  There the latency of a block
// counts, and the second path for waves of interior cells lengthens it; with
// more blocks the even-odd form wins by its registers, which let two blocks
// share a CU (degree 8) or three.  Four sweeps, plain against even-odd: degree
// 7, 7^2 cells 29 against 35 us, 120^2 52 against 54, 150^2 80 against 68;
// degree 8, 64^2 41.6 against 44.1, 90^2 74 against 57; degree 6, 50^2 30 against
// 34, 150^2 70 against 57.
#define HPMG_TILE 4
#include "dg_inst.hpp"

namespace hpmg {
namespace {
template <int N>
bool run_plain(int op, const DGArgs<double>& a, int nrhs, int flag, hipStream_t s) {
  switch (op) {
    case OP_SWEEP: return dgk_t4::launch_sweep<double, 2, N>(a, nrhs, flag != 0, s);
    case OP_APPLY: return dgk_t4::launch_apply<double, 2, N, 0>(a, nrhs, flag != 0, s);
    case OP_RESTRICT: return dgk_t4::launch_apply_r<double, 2, N, nc_next(N), true>(a, nrhs, s);
    case OP_RESTRICT_Q1: return dgk_t4::launch_apply_r<double, 2, N, 2, true>(a, nrhs, s);
    case OP_RESTRICT_DYN: return dgk_t4::launch_apply_r<double, 2, N, -1, true>(a, nrhs, s);
    default: return false;
  }
}
}  // namespace

bool dg_dispatch2_plain(int N, int op, const DGArgs<double>& a, int nrhs, int flag, hipStream_t s) {
  // blocks held at once: one per CU at degree 8 (one wave per SIMD), two below
  const int cpb = cells_per_block_v(2, N, 0);
  const long long blocks = (long long)((a.ncell + cpb - 1) / cpb) * nrhs;
  if (N < 7 || a.vark || blocks > 256 * (N == 9 ? 1 : 2)) return false;
  switch (N) {
    case 7: return run_plain<7>(op, a, nrhs, flag, s);
    case 8: return run_plain<8>(op, a, nrhs, flag, s);
    default: return run_plain<9>(op, a, nrhs, flag, s);
  }
}
}  // namespace hpmg
