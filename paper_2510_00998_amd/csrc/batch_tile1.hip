// The batched DG kernels with half the cells per block (tile variant 1 of the
// autotuner): one degree each, and all degrees at once (full bricks leave that
// one's small batches too few workgroups: 6 problems of 7^3 to 13^3 cells, degree
// 1 to 3, FP32, a projection and two sweeps 32 us, 38 with full bricks).
#define HPMG_TILE 1
#include "batch_dg_all.hpp"
