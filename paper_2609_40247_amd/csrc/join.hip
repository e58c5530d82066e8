// Launch <-> kernel join: kernels and their launches.
#include "join.hpp"

namespace hx {

template <int IT>
__global__ __launch_bounds__(256) void k_jt_store(JoinArgs a) {
  jt_store_body<IT>(a, blockIdx.x);
}

template <int IT>
__global__ __launch_bounds__(256) void k_jt_resolve(JoinArgs a) {
  __shared__ JtResolveLds lds;
  jt_resolve_body<IT>(a, lds, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_jt_dups(JoinArgs a) {
  jt_dups_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_jt_fix(JoinArgs a) {
  __shared__ JtFixLds lds;
  jt_fix_body(a, lds, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_edges(JoinArgs a) {
  edges_body(a, blockIdx.x, gridDim.x);
}

// The join after the plan and the emptied table (both from the histogram
// kernel): store, resolve and the two fix-up passes.
void launch_join_table(Ctx& c) {
  if (c.n == 0) return;
  JoinArgs a = join_args(c);
  auto grid = [&](int it) { return dim3((unsigned)jt_blocks(c, it)); };
  hipLaunchKernelGGL(k_jt_store<JT_IT_STORE>, grid(JT_IT_STORE), dim3(256), 0, c.st, a);
  hipLaunchKernelGGL(k_jt_resolve<JT_IT_RESOLVE>, grid(JT_IT_RESOLVE), dim3(256), 0, c.st, a);
  const unsigned fb = (unsigned)jt_fix_blocks(c);
  hipLaunchKernelGGL(k_jt_dups, dim3(fb), dim3(256), 0, c.st, a);
  hipLaunchKernelGGL(k_jt_fix, dim3(fb), dim3(256), 0, c.st, a);
}

void launch_edges(Ctx& c) {
  if (c.p.n_edges <= 0) return;
  JoinArgs a = join_args(c);
  const int grid = (int)std::min<int64_t>(cdiv(c.p.n_edges, 256), 1024);
  hipLaunchKernelGGL(k_edges, dim3(grid), dim3(256), 0, c.st, a);
}

}  // namespace hx
