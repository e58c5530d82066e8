// Cross-stream overlap: kernels and their launches.
#include "overlap.hpp"

namespace hx {

__global__ __launch_bounds__(256) void k_segoff(SweepArgs a) {
  segoff_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(SW_THREADS) void k_sweep_groups(SweepArgs a) {
  __shared__ SweepGroupsLds lds;
  sweep_groups_body<SW_ITEMS>(a, lds, blockIdx.x);
}

__global__ __launch_bounds__(SM_THREADS) void k_sweep_many(SweepArgs a) {
  extern __shared__ unsigned long long s_pair[];
  __shared__ SweepManyLds lds;
  sweep_many_body(a, lds, s_pair, blockIdx.x, gridDim.x);
}

void launch_overlap(Ctx& c) {
  const SweepArgs a = sweep_args(c);
  hipLaunchKernelGGL(k_segoff, dim3((unsigned)segoff_blocks(c)), dim3(256), 0, c.st, a);
  if (sweep_by_groups(c))
    hipLaunchKernelGGL(k_sweep_groups, dim3((unsigned)sweep_groups_blocks(c, SW_ITEMS)), dim3(SW_THREADS), 0, c.st, a);
  else
    hipLaunchKernelGGL(k_sweep_many, dim3((unsigned)sweep_many_blocks(c)), dim3(SM_THREADS), (size_t)c.S * c.S * 8,
                       c.st, a);
}

}  // namespace hx
