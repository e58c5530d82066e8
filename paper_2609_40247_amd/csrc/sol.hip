// Operator efficiency: kernels and their launches.
#include "sol.hpp"

namespace hx {

__global__ __launch_bounds__(SOL_THREADS) void k_sol(SolArgs a) {
  extern __shared__ unsigned long long tab[];
  sol_body(a, tab, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_sol_fold(SolArgs a, int blocks) {
  sol_fold_body(a, blocks, blockIdx.x, blockIdx.y, gridDim.y);
}

__global__ __launch_bounds__(256) void k_sol_names(SolArgs a) {
  sol_names_body(a, blockIdx.x);
}

// Workgroups of the op pass: about 2048 rows each, at most SOL_MAX_BLOCKS,
// and with name tables no more than SOL_PART_BYTES of them.
int sol_block_count(int64_t n_max, int NOP) {
  int64_t b = std::min<int64_t>(cdiv(n_max, 2048), SOL_MAX_BLOCKS);
  if (sol_uses_tables(NOP)) b = std::min<int64_t>(b, SOL_PART_BYTES / ((int64_t)NOP * 32));
  return (int)std::max<int64_t>(b, 1);
}

bool sol_uses_tables(int NOP) { return NOP <= SOL_LDS_NAMES; }

void launch_sol(Ctx& c) {
  SolArgs a = sol_args(c);
  const size_t lds = a.lds ? (size_t)c.NOP * 32 : 0;
  hipLaunchKernelGGL(k_sol, dim3((unsigned)c.sol_blocks), dim3(SOL_THREADS), lds, c.st, a);
  if (a.lds) {
    const unsigned gx = (unsigned)cdiv((int64_t)c.NOP * 4, 256);
    const unsigned gy = (unsigned)std::min(SF_ROWS, c.sol_blocks);
    hipLaunchKernelGGL(k_sol_fold, dim3(gx, gy), dim3(256), 0, c.st, a, c.sol_blocks);
  }
  hipLaunchKernelGGL(k_sol_names, dim3((unsigned)cdiv(c.NOP, 256)), dim3(256), 0, c.st, a);
}

}  // namespace hx
