// Instantiation of the DG cell kernels for dim = 3, storage type double: variable kappa.
#define HPMG_TILE 2
#include "dg_inst.hpp"

namespace hpmg {
bool dg_dispatch3_vark(int N, int op, const DGArgs<double>& a, int nrhs, int flag, hipStream_t s) {
  return dgk_t2::dispatch<double, 3>(N, op, a, nrhs, flag, s);
}
}  // namespace hpmg
