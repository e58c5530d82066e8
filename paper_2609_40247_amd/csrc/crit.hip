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

__global__ __launch_bounds__(256) void k_crit_far_walk(CritArgs a) {
  crit_far_walk_body(a, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_crit_far_fill(CritArgs a) {
  crit_far_fill_body(a, blockIdx.x, gridDim.x);
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

static void launch_crit_marks(Ctx& c, CritArgs a, uint32_t left) {
  a.left = left;
  hipLaunchKernelGGL(k_crit_mark_local, dim3((unsigned)cdiv(2 * c.n, CP_TE)), dim3(CP_MLT), 0, c.st, a);
  hipLaunchKernelGGL(k_crit_attr, dim3(crit_grid(c.n)), dim3(256), 0, c.st, a);
}

// The pointers of level l, 32 steps of the level below.  Those of a small
// window stay in the caches: one launch follows all 32 (28 us for 400k events).
// Beyond, the gathers count: jumps of 4, 4 and 2 (seven gathers an event), and
// of many events five squarings (five gathers, two launches more; critical
// paths of shuffled traces of 1.5M rows, squarings and 4-4-2, 824 / 829 us a
// call and 872 / 856 a window of a batch, of 3.0M rows 1467 / 1516 and 1525 /
// 1558).
constexpr int64_t CP_SQUARE_EVENTS = 1 << 22;

static void launch_crit_level(Ctx& c, CritArgs a, int l) {
  // the kernel ends' two row buffers follow one another: [2n] words between them
  int32_t* const tmp = reinterpret_cast<int32_t*>(c.sE.v[0]);
  const unsigned grid = c.small ? (unsigned)cdiv(2 * c.n, 256) : crit_grid(2 * c.n);
  static constexpr int once[] = {CP_STRIDE, 0}, three[] = {4, 4, 2, 0}, squares[] = {2, 2, 2, 2, 2, 0};
  a.jump_in = a.lv[l - 1];
  a.jump_out = a.lv[l];  // an odd number of jumps ends there
  for (const int* st = c.small ? once : 2 * c.n <= CP_SQUARE_EVENTS ? three : squares; *st; ++st) {
    a.jump_steps = *st;
    hipLaunchKernelGGL(k_crit_jump, dim3(grid), dim3(256), 0, c.st, a);
    a.jump_in = a.jump_out;
    a.jump_out = a.jump_out == tmp ? a.lv[l] : tmp;
  }
}

// The strides, and where they stop short the further levels.
static void launch_crit_strides(Ctx& c, CritArgs a) {
  a.need = CP_MORE_STRIDES;
  launch_crit_level(c, a, 1);
  hipLaunchKernelGGL(k_crit_strides, dim3((unsigned)std::min(c.P, 2048)), dim3(CP_HOPS), 0, c.st, a);
}
static void launch_crit_far(Ctx& c, CritArgs a) {
  a.need = CP_MORE_FAR;
  for (int l = 2; l <= a.levels; ++l) launch_crit_level(c, a, l);
  hipLaunchKernelGGL(k_crit_far_walk, dim3((unsigned)cdiv(c.P, 256)), dim3(256), 0, c.st, a);
  const unsigned grid = (unsigned)std::min<int64_t>(cdiv(2 * c.n, 256), 1 << 20);
  for (a.fill = a.levels; a.fill > 0; --a.fill)
    hipLaunchKernelGGL(k_crit_far_fill, dim3(grid), dim3(256), 0, c.st, a);
}

// With c.crit_deferred the further levels, and but for small windows the
// strides, are left out: the charging pass then does nothing if a walk stopped
// short (DevState::crit_more), and the caller runs launch_crit_deferred once
// the call has ended.  (A small window's strides are two launches, about 2 us
// each when they have nothing to do and a round trip to the host less when
// they have.)
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
    launch_crit_strides(c, a);
    launch_crit_far(c, a);
    launch_crit_marks(c, a, 0);
    return;
  }
  if (c.small) {
    launch_crit_strides(c, a);
    launch_crit_marks(c, a, CP_MORE_FAR);
  } else {
    launch_crit_marks(c, a, CP_MORE_STRIDES | CP_MORE_FAR);
  }
}

void launch_crit_deferred(Ctx& c, bool far) {
  if (c.n == 0) return;
  CritArgs a = crit_args(c);
  if (far) {
    launch_crit_far(c, a);
    launch_crit_marks(c, a, 0);
  } else {
    launch_crit_strides(c, a);
    launch_crit_marks(c, a, CP_MORE_FAR);
  }
}

}  // namespace hx
