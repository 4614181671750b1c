// The one-degree batched DG kernels with half the cells per block (tile
// variant 1 of the autotuner), and the kernel that takes all degrees at once.
#define HPMG_TILE 1
#include "batch_dg_body.hpp"

// One launch over all degrees, in the cell blocks of variant 1: small batches,
// whose launches take longer than their work, gain from one launch per step,
// and the full blocks leave them too few workgroups (6 problems of 7^3 to 13^3
// cells, degree 1 to 3, FP32, a projection and two sweeps: 29 us in cell runs,
// 38 with full bricks, 32 here).
namespace hpmg {
namespace {

constexpr int cmax(int a, int b) { return a > b ? a : b; }

template <typename T, int OP>
constexpr int batch_lds() {
  return cmax(cmax(cmax(item_lds<T, 2, OP>(), item_lds<T, 3, OP>()), cmax(item_lds<T, 4, OP>(), item_lds<T, 5, OP>())),
              item_lds<T, 6, OP>());
}

// threads of a block that takes items of any degree
constexpr int BATCH_BLOCK = cmax(cmax(cmax(DGShapeV<3, 2, 1>::BLOCK, DGShapeV<3, 3, 1>::BLOCK),
                                      cmax(DGShapeV<3, 4, 1>::BLOCK, DGShapeV<3, 5, 1>::BLOCK)),
                                 DGShapeV<3, 6, 1>::BLOCK);

template <typename T, int OP>
__global__ __launch_bounds__(BATCH_BLOCK) void k_dg_batch(const DGArgs<T>* __restrict__ args,
                                                  const WorkItem* __restrict__ items, int nitems) {
  __shared__ __attribute__((aligned(16))) char lds[batch_lds<T, OP>()];
  for (int it = blockIdx.x; it < nitems; it += gridDim.x) {
    const WorkItem w = items[it];
    const DGArgs<T> a = args[w.x];
    switch (w.w) {
      case 2: dg_item<T, 2, OP>(a, w.y, w.z, lds); break;
      case 3: dg_item<T, 3, OP>(a, w.y, w.z, lds); break;
      case 4: dg_item<T, 4, OP>(a, w.y, w.z, lds); break;
      case 5: dg_item<T, 5, OP>(a, w.y, w.z, lds); break;
      case 6: dg_item<T, 6, OP>(a, w.y, w.z, lds); break;
      default: break;
    }
    __syncthreads();  // the next item reuses the LDS
  }
}

}  // namespace

template <typename T>
void batch_dg(int op, const DGArgs<T>* args, const WorkItem* items, int nitems, int grid, hipStream_t s) {
  const dim3 g(grid_for_n(nitems, grid)), b(BATCH_BLOCK);
  switch (op) {
    case BOP_SWEEP: hipLaunchKernelGGL((k_dg_batch<T, BOP_SWEEP>), g, b, 0, s, args, items, nitems); break;
    case BOP_SWEEP0: hipLaunchKernelGGL((k_dg_batch<T, BOP_SWEEP0>), g, b, 0, s, args, items, nitems); break;
    case BOP_RESTRICT: hipLaunchKernelGGL((k_dg_batch<T, BOP_RESTRICT>), g, b, 0, s, args, items, nitems); break;
    case BOP_PROLONG: hipLaunchKernelGGL((k_dg_batch<T, BOP_PROLONG>), g, b, 0, s, args, items, nitems); break;
    case BOP_PROJECT: hipLaunchKernelGGL((k_dg_batch<T, BOP_PROJECT>), g, b, 0, s, args, items, nitems); break;
    case BOP_RESID: hipLaunchKernelGGL((k_dg_batch<T, BOP_RESID>), g, b, 0, s, args, items, nitems); break;
    default: hipLaunchKernelGGL((k_dg_batch<T, BOP_APPLY>), g, b, 0, s, args, items, nitems); break;
  }
}

template void batch_dg<float>(int, const DGArgs<float>*, const WorkItem*, int, int, hipStream_t);
template void batch_dg<double>(int, const DGArgs<double>*, const WorkItem*, int, int, hipStream_t);

}  // namespace hpmg
