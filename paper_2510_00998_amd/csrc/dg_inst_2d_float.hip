// Instantiation of the DG cell kernels for dim = 2, storage type float.
#include "dg_inst.hpp"

namespace hpmg {
bool dg_dispatch2(int N, int op, const DGArgs<float>& a, int nrhs, int flag, hipStream_t s) {
  return dgk::dispatch<float, 2>(N, op, a, nrhs, flag, s);
}
}  // namespace hpmg
