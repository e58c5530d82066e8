// Radix sort: kernels and their launches.
#include "radix.hpp"

namespace hx {

__global__ __launch_bounds__(HIST_THREADS) void k_digit_hist(HistJobs jobs, DevState* ds) {
  __shared__ DigitHistLds lds;
  digit_hist_body(jobs, ds, lds, blockIdx.x, blockIdx.y, gridDim.x);
}

__global__ __launch_bounds__(PLAN_THREADS) void k_hist_plan(HistJobs jobs, DevState* ds) {
  __shared__ HistPlanLds lds;
  hist_plan_body(jobs, ds, lds, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(RS_THREADS) __attribute__((amdgpu_waves_per_eu(RS_WAVES_PER_EU))) void k_radix_pass(SortJobs jobs, DevState* ds) {
  __shared__ RadixPassLds<false> lds;
  radix_pass_body<false>(jobs, ds, lds, blockIdx.x);
}

__global__ __launch_bounds__(RS_THREADS) __attribute__((amdgpu_waves_per_eu(RS_PK_WAVES_PER_EU))) void k_radix_pass_packed(SortJobs jobs, DevState* ds) {
  __shared__ RadixPassLds<true> lds;
  radix_pass_body<true>(jobs, ds, lds, blockIdx.x);
}

template <bool PACKED>
__global__ __launch_bounds__(RF_THREADS) void k_refine(RefineJobs jobs, DevState* ds) {
  __shared__ RefineLds lds;
  refine_body<PACKED>(jobs, ds, lds, blockIdx.x, blockIdx.y);
}

void launch_hist_multi(Ctx& c, SortBufs* const* s, const int32_t* const* count, int k) {
  int64_t grid;
  int m, nd;
  const HistJobs jobs = hist_jobs(c, s, count, k, &grid, &m, &nd);
  hipLaunchKernelGGL(k_digit_hist, dim3((unsigned)grid, (unsigned)(m + 1)), dim3(HIST_THREADS), 0, c.st, jobs,
                     c.ds);
  if (m > 0)
    hipLaunchKernelGGL(k_hist_plan, dim3((unsigned)nd, (unsigned)m), dim3(PLAN_THREADS), 0, c.st, jobs, c.ds);
}

// Passes p0 .. p1-1 of up to N_SORTS sorts, one launch per pass.
void launch_sort_multi(Ctx& c, SortBufs* const* s, const int32_t* const* count, int k, int p0, int p1) {
  for (int p = p0; p < p1; ++p) {
    int64_t grid;
    const SortJobs jobs = sort_jobs(c, s, count, k, p, &grid);
    if (jobs.m == 0) continue;
    hipLaunchKernelGGL(c.packed ? k_radix_pass_packed : k_radix_pass, dim3((unsigned)grid), dim3(RS_THREADS), 0, c.st, jobs, c.ds);
  }
}

void launch_refine(Ctx& c) {
  int64_t grid;
  int m;
  const RefineJobs jobs = refine_jobs(c, &grid, &m);
  if (m == 0) return;
  hipLaunchKernelGGL(c.packed ? k_refine<true> : k_refine<false>, dim3((unsigned)grid, (unsigned)m), dim3(RF_THREADS), 0, c.st, jobs, c.ds);
}

}  // namespace hx
