// One launch over all degrees of a batch, in the cell blocks of HPMG_TILE (see
// batch_dg_body.hpp): small batches, whose launches take longer than their
// work, gain from one launch per step.
#pragma once
#include "batch_dg_body.hpp"

#define HPMG_BATCH_DG_ALL HPMG_BATCH_CAT(batch_dg_t, HPMG_TILE)

namespace hpmg {
namespace {

constexpr int cmax(int a, int b) { return a > b ? a : b; }

template <typename T, int OP>
constexpr int batch_lds() {
  return cmax(cmax(cmax(item_lds<T, 2, OP>(), item_lds<T, 3, OP>()), cmax(item_lds<T, 4, OP>(), item_lds<T, 5, OP>())),
              item_lds<T, 6, OP>());
}

// threads of a block that takes items of any degree
constexpr int BATCH_BLOCK = cmax(cmax(cmax(DGShapeV<3, 2, HPMG_TILE>::BLOCK, DGShapeV<3, 3, HPMG_TILE>::BLOCK),
                                      cmax(DGShapeV<3, 4, HPMG_TILE>::BLOCK, DGShapeV<3, 5, HPMG_TILE>::BLOCK)),
                                 DGShapeV<3, 6, HPMG_TILE>::BLOCK);

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
void HPMG_BATCH_DG_ALL(int op, const DGArgs<T>* args, const WorkItem* items, int nitems, int grid, hipStream_t s) {
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

template void HPMG_BATCH_DG_ALL<float>(int, const DGArgs<float>*, const WorkItem*, int, int, hipStream_t);
template void HPMG_BATCH_DG_ALL<double>(int, const DGArgs<double>*, const WorkItem*, int, int, hipStream_t);

}  // namespace hpmg
