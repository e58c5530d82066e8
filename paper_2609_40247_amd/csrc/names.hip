// Per-name tables: kernels and their launches.
#include "names.hpp"

namespace hx {

__global__ __launch_bounds__(NM_THREADS) void k_names_partial(NamesArgs a) {
  extern __shared__ unsigned long long tab[];
  names_partial_body(a, tab, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(KO_THREADS) void k_kernel_ops(NamesArgs a) {
  kernel_ops_body(a, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_names_reduce(NamesArgs a) {
  names_reduce_body(a, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(ON_THREADS) void k_opnames_partial(OpNamesArgs a) {
  extern __shared__ unsigned long long otab[];
  opnames_partial_body(a, otab, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_opnames_fold(OpNamesArgs a) {
  opnames_fold_body(a, blockIdx.x, blockIdx.y, gridDim.y);
}

int names_block_count(int64_t n_max, int NN) {
  if (NN > NM_LDS_NAMES) return (int)std::min<int64_t>(std::max<int64_t>(cdiv(n_max, 4096), 1), 1024);
  // small windows: 4096 rows a workgroup, unless the tables get large
  const int64_t b = std::max(NN <= 2048 ? cdiv(std::min(n_max, SMALL_ROWS), 4096) : 0, cdiv(n_max, 8192));
  return (int)std::min<int64_t>(std::max<int64_t>(b, 1), 256);
}

void launch_names(Ctx& c) {
  if (!names_wanted(c)) return;
  NamesArgs a = names_args(c);
  const size_t lds = c.NN <= NM_LDS_NAMES ? (size_t)c.NN * 32 : 0;
  hipLaunchKernelGGL(k_names_partial, dim3(c.name_blocks), dim3(NM_THREADS), lds, c.st, a);
}

// after the join and the containment query
void launch_kernel_ops(Ctx& c) {
  if (!c.contain) return;
  NamesArgs a = names_args(c);
  hipLaunchKernelGGL(k_kernel_ops, dim3((unsigned)kernel_ops_blocks(c)), dim3(KO_THREADS), 0, c.st, a);
}

void launch_names_reduce(Ctx& c) {
  if (c.NN > NM_LDS_NAMES || !names_wanted(c)) return;
  NamesArgs a = names_args(c);
  hipLaunchKernelGGL(k_names_reduce, dim3((unsigned)cdiv((int64_t)c.NN * 4, 256), (unsigned)names_fold_rows(c)), dim3(256),
                     0, c.st, a);
}

bool opnames_use_tables(int NOP) { return NOP <= ON_LDS_NAMES; }
// one workgroup per 4096 entries, capped at ON_MAX_BLOCKS and so that the
// per-workgroup tables (NOP * 32 bytes each) stay within 4 MB
int opnames_block_count(int64_t n_max, int NOP) {
  const int64_t cap = std::max<int64_t>((int64_t)(4 << 20) / ((int64_t)std::max(NOP, 1) * 32), 1);
  return (int)std::min<int64_t>({std::max<int64_t>(cdiv(n_max, 4096), 1), (int64_t)ON_MAX_BLOCKS, cap});
}

void launch_opnames(Ctx& c) {
  if (!opnames_wanted(c) || c.n == 0) return;
  const OpNamesArgs a = opnames_args(c);
  hipLaunchKernelGGL(k_opnames_partial, dim3((unsigned)c.opn_blocks), dim3(ON_THREADS),
                     a.lds ? (size_t)c.NOP * 32 : 0, c.st, a);
  if (a.lds) {
    const unsigned gy = (unsigned)opnames_fold_rows(c);
    hipLaunchKernelGGL(k_opnames_fold, dim3((unsigned)cdiv((int64_t)c.NOP * 4, 256), gy), dim3(256), 0, c.st, a);
  }
}

int names_lds_limit() { return NM_LDS_NAMES; }

hipError_t names_set_lds_attr() {
  return hipFuncSetAttribute((const void*)k_names_partial, hipFuncAttributeMaxDynamicSharedMemorySize,
                             NM_LDS_NAMES * 32);
}

}  // namespace hx
