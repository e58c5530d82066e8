// Containment: kernels and their launches.
#include "contain.hpp"

namespace hx {

__global__ __launch_bounds__(VB_THREADS) void k_vbuild(ContainArgs a) {
  __shared__ VbuildLds lds;
  vbuild_body(a, lds, blockIdx.x);
}

__global__ __launch_bounds__(QY_THREADS) void k_query(ContainArgs a) {
  __shared__ QueryLds lds;
  query_body(a, lds, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_depth(ContainArgs a) {
  __shared__ DepthLds lds;
  depth_body(a, lds, blockIdx.x);
}

__global__ __launch_bounds__(AG_THREADS) void k_opagg(ContainArgs a) {
  __shared__ OpaggLds lds;
  opagg_body(a, lds, blockIdx.x);
}

void launch_contain(Ctx& c) {
  ContainArgs a = contain_args(c);
  const int64_t tiles = std::max<int64_t>(cdiv(c.sC.n_max, CT_TILE), 1);
  hipLaunchKernelGGL(k_vbuild, dim3((unsigned)tiles), dim3(VB_THREADS), 0, c.st, a);
  hipLaunchKernelGGL(k_query, dim3((unsigned)tiles), dim3(QY_THREADS), 0, c.st, a);
}

void launch_depth(Ctx& c) {
  ContainArgs a = contain_args(c);
  hipLaunchKernelGGL(k_depth, dim3((unsigned)std::max<int64_t>(cdiv(c.sC.n_max, 256 * DP_ITEMS), 1)), dim3(256), 0,
                     c.st, a);
}

void launch_opagg(Ctx& c) {
  ContainArgs a = contain_args(c);
  const int64_t tiles = std::max<int64_t>(cdiv(c.sC.n_max, AG_TILE), 1);
  hipLaunchKernelGGL(k_opagg, dim3((unsigned)tiles), dim3(AG_THREADS), 0, c.st, a);
}

}  // namespace hx
