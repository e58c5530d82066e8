// The first and the last kernel of a call: kernels and their launches.
#include "frame.hpp"

namespace hx {

__global__ __launch_bounds__(256) void k_init(InitArgs a) {
  init_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_nocontain(const uint64_t* keys, const uint32_t* rows, DevState* ds, int32_t* link, int32_t* aux) {
  nocontain_body(keys, rows, ds, link, aux, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_finalize(DevState* ds, herschel_counters* cnt, int64_t* lat_hist, const int64_t* busy, int64_t* idle, int nps, int64_t W, Mailbox* mb, int64_t seq) {
  finalize_body(ds, cnt, lat_hist, busy, idle, nps, W, mb, seq);
}

void launch_init(Ctx& c) {
  const InitArgs a = init_args(c);
  hipLaunchKernelGGL(k_init, dim3((unsigned)init_blocks(c, a)), dim3(256), 0, c.st, a);
}

void launch_nocontain(Ctx& c) {
  const int grid = (int)std::min<int64_t>(std::max<int64_t>(cdiv(c.n, 256 * 8), 1), 2048);
  hipLaunchKernelGGL(k_nocontain, dim3(grid), dim3(256), 0, c.st, c.sC.k[0], c.sC.v[0], c.ds, c.o.link, c.o.aux);
}

void launch_finalize(Ctx& c) {
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, c.st, c.ds, c.o.counters, c.o.lat_hist,
                     c.o.busy ? c.o.busy : c.busy_ws, c.o.idle, c.P * c.S, c.W, c.mailbox, c.mailbox_seq);
}

}  // namespace hx
