// Shared body of the per-(type, dimension, block shape) instantiation files:
// dispatch of a DG operation to the kernel of degree N - 1.
#pragma once
#include "dg_kernels_impl.hpp"
#include "kernels.hpp"

namespace hpmg {
namespace HPMG_DGK {

template <typename T, int D, int N>
bool run(int op, const DGArgs<T>& a, int nrhs, int flag, hipStream_t s) {
  constexpr int NC = nc_next(N);
  switch (op) {
    case OP_SWEEP: return launch_sweep<T, D, N>(a, nrhs, flag != 0, s);
    case OP_APPLY: return launch_apply<T, D, N, 0>(a, nrhs, flag != 0, s);
    case OP_RESTRICT: return launch_apply_r<T, D, N, NC, true>(a, nrhs, s);
    case OP_PROJECT: return launch_prolong<T, D, N, 0>(a, nrhs, s);
    case OP_PROLONG: return launch_prolong<T, D, N, NC>(a, nrhs, s);
    case OP_RESTRICT_Q1: return launch_apply_r<T, D, N, 2, true>(a, nrhs, s);
    case OP_PROLONG_Q1: return launch_prolong<T, D, N, 2>(a, nrhs, s);
    case OP_RESTRICT_DYN:
      if constexpr (N >= 4) return launch_apply_r<T, D, N, -1, true>(a, nrhs, s);
      return false;
    case OP_PROLONG_DYN:
      if constexpr (N >= 4) return launch_prolong<T, D, N, -1>(a, nrhs, s);
      return false;
    case OP_BUILD_EIG:
      if constexpr (std::is_same<T, double>::value || std::is_same<T, float>::value)
        return launch_build_eig<T, D, N>(a, s);
      return false;
    default: return false;
  }
}

template <typename T, int D>
bool dispatch(int N, int op, const DGArgs<T>& a, int nrhs, int flag, hipStream_t s) {
  switch (N) {
    case 2: return run<T, D, 2>(op, a, nrhs, flag, s);
    case 3: return run<T, D, 3>(op, a, nrhs, flag, s);
    case 4: return run<T, D, 4>(op, a, nrhs, flag, s);
    case 5: return run<T, D, 5>(op, a, nrhs, flag, s);
    case 6: return run<T, D, 6>(op, a, nrhs, flag, s);
    case 7: return run<T, D, 7>(op, a, nrhs, flag, s);
    case 8: return run<T, D, 8>(op, a, nrhs, flag, s);
    case 9: return run<T, D, 9>(op, a, nrhs, flag, s);
    default: return false;
  }
}

}  // namespace HPMG_DGK
}  // namespace hpmg
