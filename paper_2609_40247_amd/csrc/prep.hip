// Prep: kernels and their launches.
#include "prep.hpp"

namespace hx {

__global__ __launch_bounds__(PREP_THREADS) void k_prep(PrepArgs a) {
  __shared__ PrepLds<PREP_ITEMS> lds;
  prep_body(a, lds, blockIdx.x);
}

void launch_prep(Ctx& c) {
  if (c.n == 0) return;
  hipLaunchKernelGGL(k_prep, dim3((unsigned)c.prep_tiles), dim3(PREP_THREADS), 0, c.st, prep_args(c));
}

int64_t prep_tile_rows(bool small) { return PREP_THREADS * (small ? PREP_ITEMS_SMALL : PREP_ITEMS); }

}  // namespace hx
