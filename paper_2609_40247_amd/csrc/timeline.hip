// Per-stream timelines: kernels and their launches.
#include "timeline.hpp"

namespace hx {

__global__ __launch_bounds__(UN_THREADS) void k_union(UnionArgs a) {
  __shared__ UnionLds<UN_THREADS> lds;
  union_body(a, lds, blockIdx.x);
}

static void launch_union(Ctx& c, const UnionArgs& a) {
  hipLaunchKernelGGL(k_union, dim3((unsigned)c.union_tiles), dim3(UN_THREADS), 0, c.st, a);
}
void launch_timeline(Ctx& c) { launch_union(c, timeline_args(c)); }
void launch_union_device(Ctx& c) { launch_union(c, union_device_args(c)); }
void launch_union_opnames(Ctx& c) { launch_union(c, union_opnames_args(c)); }

int64_t union_tile_elems(bool small) { return (small ? UN_THREADS_SMALL : UN_THREADS) * UN_ITEMS; }

}  // namespace hx
