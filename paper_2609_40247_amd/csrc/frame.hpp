// The first and the last kernel of a call: clearing, and the counters.
#pragma once

#include "internal.hpp"

#include <cstddef>

namespace hx {

struct InitArgs {
  DevState* ds;
  uint4* zero;
  int64_t zero_n;  // 16-byte words
  herschel_counters* cnt;
  int64_t* busy;
  int nps;
  int64_t* lat_hist;
  bool overlap;
  int64_t* pair;
  int64_t* class_busy;
  int64_t* class_overlap;
  int64_t* any_busy;
  int P, S;
  int NN;
  int64_t* name_count;
  int64_t* name_sum;
  int64_t* name_min;
  int64_t* name_max;
  const int64_t* off;
  const uint8_t* cls;
  int64_t n_opn;      // P * n_op_names with the idle-coincidence outputs, else 0
  int64_t n_crit;     // P * 8 with the critical path, else 0
  int64_t* crit_proc;
  int NOP;
  int64_t* opn[4];    // per op name: count, sum, min, max (each may be NULL)
  int64_t n_gn;       // graph nodes with the graph replay outputs, else 0
  int64_t* gn[5];     // count, sum, min, max, offset (each may be NULL)
  int64_t* op_span;
  int64_t* op_idle;
};

// The device state is cleared up to its digit offsets (the plan kernel
// writes those whole, after this; the last 16-byte word may reach into
// them), 16 bytes a thread over the grid; the word of the smallest invalid
// row starts at INT64_MAX.  The status word lies in the first workgroup's
// share, so its parameter check follows the clearing.
constexpr int64_t DS_CLEAR = ((int64_t)offsetof(DevState, hist) + 15) / 16;
constexpr int64_t DS_FI = (int64_t)offsetof(DevState, first_invalid);
static_assert(DS_CLEAR * 16 <= (int64_t)sizeof(DevState) && DS_FI % 8 == 0, "16-byte clearing of the device state");
static_assert(alignof(DevState) >= 8, "the device state starts the 256-byte aligned workspace");
static_assert(offsetof(DevState, status) < 256 * 16, "the status word is cleared by the first workgroup");

__device__ __forceinline__ void init_body(const InitArgs& a, uint32_t bx, uint32_t gx) {
  const int64_t tid = (int64_t)bx * 256 + threadIdx.x, nth = (int64_t)gx * 256;
  for (int64_t i = tid; i < a.zero_n; i += nth) a.zero[i] = make_uint4(0, 0, 0, 0);
  for (int64_t i = tid; i < DS_CLEAR; i += nth) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (i == DS_FI / 16) {
      if (DS_FI % 16 == 0) {
        v.x = 0xffffffffu;
        v.y = 0x7fffffffu;
      } else {
        v.z = 0xffffffffu;
        v.w = 0x7fffffffu;
      }
    }
    reinterpret_cast<uint4*>(a.ds)[i] = v;
  }
  if (bx == 0) {
    __syncthreads();
    int64_t* cz = (int64_t*)a.cnt;
    for (int i = threadIdx.x; i < (int)(sizeof(herschel_counters) / 8); i += 256) cz[i] = 0;
    if (a.lat_hist && threadIdx.x < 64) a.lat_hist[threadIdx.x] = 0;
    bool bad = false;
    if (a.off)
      for (int q = threadIdx.x; q < a.P; q += 256)
        bad |= !(a.off[q] > -HERSCHEL_MAX_ABS_TIME && a.off[q] < HERSCHEL_MAX_ABS_TIME);
    if (a.cls)
      for (int s = threadIdx.x; s < a.S; s += 256) bad |= a.cls[s] > 2;
    if (bad) atomicOr(&a.ds->status, DS_PARAM);
  }
  for (int64_t i = tid; i < a.nps; i += nth) a.busy[i] = 0;
  if (a.overlap) {
    if (a.pair)
      for (int64_t i = tid; i < (int64_t)a.nps * a.S; i += nth) a.pair[i] = 0;
    if (a.class_busy)
      for (int64_t i = tid; i < (int64_t)a.P * 3; i += nth) a.class_busy[i] = 0;
    if (a.class_overlap)
      for (int64_t i = tid; i < (int64_t)a.P * 9; i += nth) a.class_overlap[i] = 0;
    if (a.any_busy)
      for (int64_t i = tid; i < a.P; i += nth) a.any_busy[i] = 0;
  }
  // the name outputs start as the identities: the per-block tables (or,
  // with many names, the kernels themselves) are combined into them with
  // atomics
  for (int64_t i = tid; i < a.n_crit; i += nth) a.crit_proc[i] = 0;  // accumulated with atomics
  for (int64_t i = tid; i < a.NOP; i += nth) {  // combined with atomics
    if (a.opn[0]) a.opn[0][i] = 0;
    if (a.opn[1]) a.opn[1][i] = 0;
    if (a.opn[2]) a.opn[2][i] = I64MAX;
    if (a.opn[3]) a.opn[3][i] = I64MIN;
  }
  for (int64_t i = tid; i < a.n_gn; i += nth) {  // combined with atomics
    if (a.gn[0]) a.gn[0][i] = 0;
    if (a.gn[1]) a.gn[1][i] = 0;
    if (a.gn[2]) a.gn[2][i] = I64MAX;
    if (a.gn[3]) a.gn[3][i] = I64MIN;
    if (a.gn[4]) a.gn[4][i] = 0;
  }
  for (int64_t i = tid; i < a.n_opn; i += nth) {  // accumulated with atomics
    if (a.op_span) a.op_span[i] = 0;
    if (a.op_idle) a.op_idle[i] = 0;
  }
  for (int64_t i = tid; i < a.NN; i += nth) {
    if (a.name_count) a.name_count[i] = 0;
    if (a.name_sum) a.name_sum[i] = 0;
    if (a.name_min) a.name_min[i] = I64MAX;
    if (a.name_max) a.name_max[i] = I64MIN;
  }
}

static inline InitArgs init_args(const Ctx& c) {
  InitArgs a;
  a.ds = c.ds;
  a.zero = (uint4*)c.zero_begin;
  a.zero_n = (int64_t)(c.zero_bytes / 16);
  a.cnt = c.o.counters;
  a.busy = c.o.busy ? c.o.busy : c.busy_ws;
  a.nps = c.P * c.S;
  a.lat_hist = c.o.lat_hist;
  a.overlap = c.overlap;
  a.pair = c.o.pair_overlap;
  a.class_busy = c.o.class_busy;
  a.class_overlap = c.o.class_overlap;
  a.any_busy = c.o.any_busy;
  a.P = c.P;
  a.S = c.S;
  a.NN = c.NN;
  a.name_count = c.o.name_count;
  a.name_sum = c.o.name_sum;
  a.name_min = c.o.name_min;
  a.name_max = c.o.name_max;
  a.off = c.p.clock_offset;
  a.cls = c.p.stream_class;
  a.n_opn = c.waits ? (int64_t)c.P * c.NOP : 0;
  a.n_crit = c.crit && c.o.crit_proc ? (int64_t)c.P * 8 : 0;
  a.crit_proc = c.o.crit_proc;
  a.NOP = c.NOP;
  a.opn[0] = c.o.opname_count;
  a.opn[1] = c.o.opname_sum;
  a.opn[2] = c.o.opname_min;
  a.opn[3] = c.o.opname_max;
  a.n_gn = c.graph ? c.NG : 0;
  a.gn[0] = c.o.gn_count;
  a.gn[1] = c.o.gn_sum;
  a.gn[2] = c.o.gn_min;
  a.gn[3] = c.o.gn_max;
  a.gn[4] = c.o.gn_offset;
  a.op_span = c.o.op_span ? c.o.op_span : c.op_span_ws;
  a.op_idle = c.o.op_idle;
  return a;
}
static inline int init_blocks(const Ctx& c, const InitArgs& a) {
  const int64_t work =
      std::max<int64_t>({a.zero_n, (int64_t)a.nps * (c.overlap ? c.S : 1), (int64_t)c.NN, a.n_opn, a.n_gn,
                         (int64_t)c.NOP, DS_CLEAR, 1});
  return (int)std::min<int64_t>(std::max<int64_t>(cdiv(work, 256 * 2), 8), 2048);
}

// Without containment, admitted ops and launches have no op links (either
// output may be NULL).
__device__ __forceinline__ void nocontain_body(const uint64_t* keys, const uint32_t* rows, DevState* ds,
                                               int32_t* link, int32_t* aux, uint32_t bx, uint32_t gx) {
  const int64_t n = ds->nCL;
  for (int64_t i = (int64_t)bx * 256 + threadIdx.x; i < n; i += (int64_t)gx * 256) {
    const uint32_t r = rows[i];
    if (link) link[r] = -1;
    if (aux && (keys[i] & 1) == 0) aux[r] = -1;
  }
}

__device__ __forceinline__ void finalize_body(DevState* ds, herschel_counters* cnt, int64_t* lat_hist,
                                              const int64_t* busy, int64_t* idle, int nps, int64_t W, Mailbox* mb,
                                              int64_t seq) {
  if (idle)
    for (int i = threadIdx.x; i < nps; i += 256) idle[i] = W - busy[i];
  // join counts and latency bins from their accumulator copies
  if (threadIdx.x < JC_N + 64) {
    unsigned long long v = 0;
#pragma unroll
    for (int k = 0; k < JOIN_COPIES; ++k) v += ds->join_acc[k][threadIdx.x];
    if (threadIdx.x >= JC_N) {
      if (v && lat_hist) lat_hist[threadIdx.x - JC_N] += (int64_t)v;
    } else {
      int64_t* dst = nullptr;
      int64_t val = (int64_t)v;
      switch (threadIdx.x) {
        case JC_MATCHED: dst = &cnt->n_matched; break;
        case JC_UNM_K: dst = &cnt->n_unmatched_kernels; break;
        case JC_DUP: dst = &cnt->n_dup_launch_corr; break;
        case JC_NEG: dst = &cnt->n_negative_latency; break;
        case JC_UNATTR: dst = &cnt->n_unattributed_kernels; break;
        default:  // JC_MLAUNCH: the unmatched launches are the others
          dst = &cnt->n_unmatched_launches;
          val = cnt->n_admitted[HERSCHEL_LAUNCH] - val;
          break;
      }
      *dst = val;
    }
  }
  if (threadIdx.x == 0) {
    cnt->first_invalid = ds->first_invalid == I64MAX ? -1 : ds->first_invalid;
    cnt->device_status = ds->status;
  }
  if (!mb) return;
  // the counters to the calling thread's mailbox, then the sequence number
  // with a release at system scope: the host that reads the number reads
  // this call's counters
  __syncthreads();
  if (threadIdx.x < (int)(sizeof(herschel_counters) / 8)) {
    const int64_t v = ((const int64_t*)cnt)[threadIdx.x];
    __hip_atomic_store(&mb->c[threadIdx.x], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (threadIdx.x == 0)
    __hip_atomic_store(&mb->crit_more, (int64_t)ds->crit_more, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  __syncthreads();
  if (threadIdx.x == 0) __hip_atomic_store(&mb->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace hx
