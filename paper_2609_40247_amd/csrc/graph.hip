// Graph replay separation: kernels and their launches.
#include "graph.hpp"

namespace hx {

__global__ __launch_bounds__(GR_THREADS) void k_graph(GraphArgs a) {
  extern __shared__ unsigned long long gtab[];
  graph_body(a, gtab, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_graph_fold(GraphArgs a) {
  graph_fold_body(a, blockIdx.x, blockIdx.y, gridDim.y);
}

bool graph_uses_tables(int NG) { return NG <= GR_LDS_NODES; }

int graph_block_count(int64_t n_max, int NG) {
  if (!graph_uses_tables(NG)) return (int)std::min<int64_t>(std::max<int64_t>(cdiv(n_max, 4096), 1), 1024);
  // small windows: 2048 rows a workgroup (25 workgroups of 8192 took 24 us on a trace of 198k rows)
  const int64_t b = std::max(cdiv(std::min(n_max, SMALL_ROWS), 2048), cdiv(n_max, 8192));
  return (int)std::min<int64_t>(std::max<int64_t>(b, 1), GR_MAX_BLOCKS);
}

void launch_graph(Ctx& c) {
  GraphArgs a = graph_args(c);
  const size_t lds = a.lds ? (size_t)c.NG * GR_STATS * 8 : 0;
  hipLaunchKernelGGL(k_graph, dim3((unsigned)c.graph_blocks), dim3(GR_THREADS), lds, c.st, a);
  if (a.lds) {
    const unsigned gy = (unsigned)graph_fold_rows(c);
    hipLaunchKernelGGL(k_graph_fold, dim3((unsigned)cdiv((int64_t)c.NG * GR_STATS, 256), gy), dim3(256), 0, c.st,
                       a);
  }
}

}  // namespace hx
