// Instantiation of the DG cell kernels for dim = 3, storage type double:
// constant kappa on all but small meshes; variable kappa, and adaptive and small
// meshes have block shapes of their own (dg_inst_3d_double_vark.hip,
// dg_inst_3d_double_runs.hip).
#include "dg_inst.hpp"

namespace hpmg {
bool dg_dispatch3(int N, int op, const DGArgs<double>& a, int nrhs, int flag, hipStream_t s) {
  if (a.adapt || (!a.vark && mesh_variant(a.n, N, true) == 3)) return dg_dispatch3_runs(N, op, a, nrhs, flag, s);
  if (a.vark) return dg_dispatch3_vark(N, op, a, nrhs, flag, s);
  return dgk::dispatch<double, 3>(N, op, a, nrhs, flag, s);
}
}  // namespace hpmg
