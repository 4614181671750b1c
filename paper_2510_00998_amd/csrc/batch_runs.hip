// The batched DG kernels on runs of cells, which take the place of the half
// bricks (tile variant 1) where every mesh of the batch is small (run_cells): 6
// problems of 7^3 to 13^3 cells, degree 1 to 3, five sweeps FP64 68 -> 45 us, FP32
// 61 -> 46; 12 of 9^3 and 10^3, degree 1 to 5, 133 -> 107 and 109 -> 88.
#define HPMG_TILE 3
#include "batch_dg_all.hpp"
