// Idle coincidence: kernels and their launches.
#include "waits.hpp"

namespace hx {

__global__ __launch_bounds__(DG_THREADS) void k_dg_scan(WaitsArgs a) {
  __shared__ DgScanLds lds;
  dg_scan_body(a, lds, blockIdx.x);
}

__global__ __launch_bounds__(WT_THREADS) void k_waits(WaitsArgs a) {
  __shared__ WaitsLds lds;
  waits_body(a, lds, blockIdx.x, gridDim.x);
}

void launch_dg_scan(Ctx& c) {
  const WaitsArgs a = waits_args(c);
  hipLaunchKernelGGL(k_dg_scan, dim3((unsigned)c.dg_tiles), dim3(DG_THREADS), 0, c.st, a);
}

void launch_waits(Ctx& c) {
  const WaitsArgs a = waits_args(c);
  hipLaunchKernelGGL(k_waits, dim3((unsigned)waits_blocks(c)), dim3(WT_THREADS), 0, c.st, a);
}

}  // namespace hx
