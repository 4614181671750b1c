// Instantiation of the DG cell kernels for dim = 3, storage type float: adaptive and small
// meshes (run_cells).
#define HPMG_TILE 3
#include "dg_inst.hpp"

namespace hpmg {
bool dg_dispatch3_runs(int N, int op, const DGArgs<float>& a, int nrhs, int flag, hipStream_t s) {
  return dgk_t3::dispatch<float, 3>(N, op, a, nrhs, flag, s);
}
}  // namespace hpmg
