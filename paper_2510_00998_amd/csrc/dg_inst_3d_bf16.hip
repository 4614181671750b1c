// Instantiation of the DG cell kernels for dim = 3, storage type __bf16.
#define HPMG_TILE 3  // runs of cells
#include "dg_inst.hpp"

namespace hpmg {
bool dg_dispatch3(int N, int op, const DGArgs<__bf16>& a, int nrhs, int flag, hipStream_t s) {
  return dgk_t3::dispatch<__bf16, 3>(N, op, a, nrhs, flag, s);
}
}  // namespace hpmg
