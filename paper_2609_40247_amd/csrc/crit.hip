// Critical path: kernels and their launches.
#include "crit.hpp"

namespace hx {

__global__ __launch_bounds__(256) void k_crit_elist(CritArgs a) {
  crit_elist_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_crit_host(CritArgs a) {
  __shared__ CritHostLds lds;
  crit_host_body(a, lds, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_crit_kernels(CritArgs a) {
  __shared__ CritKernelsLds lds;
  crit_kernels_body(a, lds, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_crit_last(CritArgs a) {
  crit_last_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_crit_ops(CritArgs a) {
  crit_ops_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_crit_rows(CritArgs a) {
  crit_rows_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(CP_LT) void k_crit_local(CritArgs a) {
  __shared__ CritLocalLds lds;
  crit_local_body(a, lds, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_crit_walk(CritArgs a) {
  crit_walk_body(a, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_crit_square(CritArgs a) {
  crit_square_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_crit_jump(CritArgs a) {
  crit_jump_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(CP_HOPS) void k_crit_strides(CritArgs a) {
  __shared__ CritStridesLds lds;
  crit_strides_body(a, lds, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(CP_MLT) void k_crit_mark_local(CritArgs a) {
  __shared__ CritMarkLocalLds lds;
  crit_mark_local_body(a, lds, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_crit_round(CritArgs a) {
  crit_round_body(a, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_crit_attr(CritArgs a) {
  __shared__ CritAttrLds lds;
  crit_attr_body(a, lds, blockIdx.x, gridDim.x);
}

void launch_crit_elist(Ctx& c) {
  if (c.n == 0) return;
  CritArgs a = crit_args(c);
  hipLaunchKernelGGL(k_crit_elist, dim3(crit_grid(c.n)), dim3(256), 0, c.st, a);
}

int crit_rounds(int64_t n) {
  int r = 1;
  while (r < CRIT_MAX_ROUNDS && ((int64_t)1 << (r - 1)) < 2 * n) ++r;
  return r;
}

static void launch_crit_marks(Ctx& c, CritArgs a, uint32_t left) {
  a.left = left;
  hipLaunchKernelGGL(k_crit_mark_local, dim3((unsigned)cdiv(2 * c.n, CP_TE)), dim3(CP_MLT), 0, c.st, a);
  hipLaunchKernelGGL(k_crit_attr, dim3(crit_grid(c.n)), dim3(256), 0, c.st, a);
}

// The strides.  The pointers of a small window stay in the caches: one launch
// follows 32 exits per event (28 us for 400k events; a round of doubling took
// 7.4 us, and these are five).
static void launch_crit_strides(Ctx& c, CritArgs a) {
  if (c.small) {
    hipLaunchKernelGGL(k_crit_jump, dim3((unsigned)cdiv(2 * c.n, 256)), dim3(256), 0, c.st, a);
  } else {
    for (a.round = 0; a.round < CP_SQUARES; ++a.round)
      hipLaunchKernelGGL(k_crit_square, dim3(crit_grid(2 * c.n)), dim3(256), 0, c.st, a);
  }
  hipLaunchKernelGGL(k_crit_strides, dim3((unsigned)std::min(c.P, 2048)), dim3(CP_HOPS), 0, c.st, a);
}

// The doubling over the exits.
static void launch_crit_rounds(Ctx& c, CritArgs a) {
  const int rounds = crit_rounds(c.n);
  for (a.round = 0; a.round < rounds; ++a.round)
    hipLaunchKernelGGL(k_crit_round, dim3(crit_grid(2 * c.n)), dim3(256), 0, c.st, a);
}

// With c.crit_deferred the doubling, and but for small windows the strides,
// are left out: the charging pass then does nothing if a walk stopped short
// (DevState::crit_more), and the caller runs launch_crit_deferred once the
// call has ended.  (A small window's strides are two launches, about 2 us each
// when they have nothing to do and a round trip to the host less when they
// have.)
void launch_crit_kernels(Ctx& c) {
  if (c.n == 0) return;
  hipLaunchKernelGGL(k_crit_kernels, dim3(crit_grid(c.n)), dim3(256), 0, c.st, crit_args(c));
}

void launch_crit_front(Ctx& c) {
  if (c.n == 0) return;
  CritArgs a = crit_args(c);
  hipLaunchKernelGGL(k_crit_host, dim3(crit_grid(c.n)), dim3(256), 0, c.st, a);
  hipLaunchKernelGGL(k_crit_last, dim3(crit_grid(c.n)), dim3(256), 0, c.st, a);
  hipLaunchKernelGGL(k_crit_ops, dim3(crit_grid(c.n)), dim3(256), 0, c.st, a);
}

void launch_crit(Ctx& c) {
  if (c.n == 0) return;
  CritArgs a = crit_args(c);
  hipLaunchKernelGGL(k_crit_rows, dim3(crit_grid(c.n)), dim3(256), 0, c.st, a);
  hipLaunchKernelGGL(k_crit_local, dim3((unsigned)cdiv(2 * c.n, CP_TE)), dim3(CP_LT), 0, c.st, a);
  launch_crit_walk(c);
}

// The walk, the marks and the charges, once every event has its exit.
void launch_crit_walk(Ctx& c) {
  if (c.n == 0) return;
  CritArgs a = crit_args(c);
  hipLaunchKernelGGL(k_crit_walk, dim3((unsigned)cdiv(c.P, 256)), dim3(256), 0, c.st, a);
  if (!c.crit_deferred) {
    // (a larger window's strides are six launches more, 13 us that nearly every
    // window of a batch would pay for nothing: straight to the doubling)
    if (c.small)
      launch_crit_strides(c, a);
    else
      a.when = CP_MORE_STRIDES;
    launch_crit_rounds(c, a);
    launch_crit_marks(c, a, 0);
    return;
  }
  if (c.small) {
    launch_crit_strides(c, a);
    launch_crit_marks(c, a, CP_MORE_DOUBLING);
  } else {
    launch_crit_marks(c, a, CP_MORE_STRIDES | CP_MORE_DOUBLING);
  }
}

void launch_crit_deferred(Ctx& c, bool doubling) {
  if (c.n == 0) return;
  CritArgs a = crit_args(c);
  if (doubling) {
    launch_crit_rounds(c, a);
    launch_crit_marks(c, a, 0);
  } else {
    launch_crit_strides(c, a);
    launch_crit_marks(c, a, CP_MORE_DOUBLING);
  }
}

}  // namespace hx
