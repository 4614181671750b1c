// Instantiation of the DG cell kernels for dim = 2, storage type double.
#include "dg_inst.hpp"

namespace hpmg {
bool dg_dispatch2(int N, int op, const DGArgs<double>& a, int nrhs, int flag, hipStream_t s) {
  return dg_dispatch2_plain(N, op, a, nrhs, flag, s) || dgk::dispatch<double, 2>(N, op, a, nrhs, flag, s);
}
}  // namespace hpmg
