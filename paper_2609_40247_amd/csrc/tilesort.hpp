// Sort of the lists of a small window in two launches, in place of the digit
// histogram, its plan, the radix passes and the refine pass (six launches
// whose few tiles leave most of the chip idle, about 50 us of the 140 of a
// 60k-row window).
//
//   tile sort: a workgroup sorts TS_TILE keys of a list in LDS (two passes of
//              the radix passes' ranking over the top bits that
//              tell the keys apart, then short runs of equal bits by counting;
//              with a longer run, passes over every bit), and writes the
//              tile and every TS_STEP-th key of it;
//   merge:     a thread per key counts, in every other tile, the keys that
//              come before it; with its place in its own tile the sum is its
//              place in the list.
//
// The merge costs a search per key and tile, which bounds the number of tiles
// (TS_TILES).
#pragma once

#include "internal.hpp"

namespace hx {

constexpr int TS_THREADS = 1024;
constexpr int TS_ITEMS = TS_TILE / TS_THREADS;
constexpr int TS_WAVES = TS_THREADS / WAVE;
constexpr int TS_STEP = TS_TILE / WAVE;  // keys between samples: a wave's lanes hold a tile's samples
static_assert(TS_ITEMS * TS_THREADS == TS_TILE && TS_THREADS >= 256, "one thread per digit value");
constexpr int TM_THREADS = 256;
static_assert(TS_TILE % TM_THREADS == 0 && TS_STEP == 64, "a workgroup's keys lie in one tile; six search steps");

struct TileSortJob {
  uint64_t* k[2];  // prep's list, and the result; the sorted tiles
  uint32_t* v[2];
  const int32_t* count;
  uint64_t* samples;  // [TS_TILES][WAVE]
  int wb;             // bits of a key below its segment (pid and stream, thread or name)
  int contain;        // 1: ops of equal key by end time down, then row
  int id;
  uint32_t b0, m0;    // the list's first workgroup in the tile sort and in the merge
};
struct TileSortJobs {
  TileSortJob j[N_SORTS];
  int m;
  const int64_t* te;
};

struct TileSortLds {
  uint64_t s_key[TS_TILE];
  uint32_t s_val[TS_TILE];
  uint32_t s_wh[TS_WAVES][256];  // per wave and digit value: counts, then places
  uint32_t s_scan[TS_WAVES];
  uint64_t s_ext[4][TS_WAVES];
};

// The bits of the tile's keys that tell them apart: segment and time, each
// from the tile's smallest on, next to each other (a key's own layout has the
// window's width between them, most of it unused by a tile).
struct TileBits {
  uint64_t seg0, t0, mask;
  int wb, tb;  // bits below the segment in a key, and here
  __device__ __forceinline__ uint64_t operator()(uint64_t k) const {
    return (((k >> wb) - seg0) << tb) | ((k & mask) - t0);
  }
};

// One stable pass over the tile by the digits dg (one per item, below 256; of
// positions from tn on 255, so that they stay last).  Item j of
// lane l is the tile's position (wave * TS_ITEMS + j) * 64 + l: items in
// order, lanes in order is the tile's order.
__device__ __forceinline__ void tile_pass(TileSortLds& lds, DevState* ds, uint64_t (&key)[TS_ITEMS],
                                          uint32_t (&val)[TS_ITEMS], const uint32_t (&dg)[TS_ITEMS]) {
  const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int p0 = wv * (TS_ITEMS * WAVE) + lane;
  auto& s_wh = lds.s_wh;
  constexpr int OR_XOR = 0xF0 | (0xCC ^ 0xAA);  // truth table of a | (b ^ c)
  for (int i = tid; i < TS_WAVES * 256; i += TS_THREADS) (&s_wh[0][0])[i] = 0;
  __syncthreads();
  uint32_t rank[TS_ITEMS];
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    uint32_t mis_lo = 0, mis_hi = 0;  // lanes with another digit
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)dg[j], q, 1);
      const uint64_t bb = __builtin_amdgcn_uicmp(m, 0u, 33);  // ballot(m != 0)
      mis_lo = __builtin_amdgcn_bitop3_b32(mis_lo, (uint32_t)bb, m, OR_XOR);
      mis_hi = __builtin_amdgcn_bitop3_b32(mis_hi, (uint32_t)(bb >> 32), m, OR_XOR);
    }
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(~mis_hi, __builtin_amdgcn_mbcnt_lo(~mis_lo, 0u));
    const uint32_t before = s_wh[wv][dg[j]];
    rank[j] = before + below;
    __builtin_amdgcn_wave_barrier();
    if (below == 0) s_wh[wv][dg[j]] = before + (uint32_t)(__builtin_popcount(~mis_lo) + __builtin_popcount(~mis_hi));
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // each digit value's count over the waves, its first place, then each wave's
  uint32_t c[TS_WAVES], tot = 0;
  if (tid < 256) {
#pragma unroll
    for (int w = 0; w < TS_WAVES; ++w) c[w] = s_wh[w][tid];
#pragma unroll
    for (int w = 0; w < TS_WAVES; ++w) tot += c[w];
  }
  uint32_t at = block_excl_sum<TS_THREADS>(tot, lds.s_scan, (uint32_t*)nullptr);
  if (tid < 256) {
#pragma unroll
    for (int w = 0; w < TS_WAVES; ++w) {
      s_wh[w][tid] = at;
      at += c[w];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    const uint32_t p = rank[j] + s_wh[wv][dg[j]];
    if (in_range(ds, p, TS_TILE)) {
      lds.s_key[p] = key[j];
      lds.s_val[p] = val[j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    key[j] = lds.s_key[p0 + j * WAVE];
    val[j] = lds.s_val[p0 + j * WAVE];
  }
}

// The tile's keys and rows to LDS, where every thread reads its neighbours'.
__device__ __forceinline__ void tile_store(TileSortLds& lds, const uint64_t (&key)[TS_ITEMS],
                                           const uint32_t (&val)[TS_ITEMS], int p0) {
  __syncthreads();  // (the passes' reads of the tile)
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    lds.s_key[p0 + j * WAVE] = key[j];
    lds.s_val[p0 + j * WAVE] = val[j];
  }
  __syncthreads();
}

// The largest of each of the workgroup's values over its waves.
template <int N>
__device__ __forceinline__ void tile_max(TileSortLds& lds, uint64_t (&x)[N]) {
  const int lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const uint64_t m = wave_allmax_u64(x[i]);
    if (lane == 0) lds.s_ext[i][wv] = m;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) x[i] = wave_allmax_u64(lane < TS_WAVES ? lds.s_ext[i][lane] : 0ull);
}

constexpr int TS_RUN = 32;  // longest run of keys equal in the bits sorted so far that is ordered by counting

__device__ __forceinline__ void tile_sort_body(const TileSortJobs& jobs, DevState* ds, TileSortLds& lds, uint32_t b) {
  int ji = 0;
  while (ji + 1 < jobs.m && b >= jobs.j[ji + 1].b0) ++ji;
  const TileSortJob& jb = jobs.j[ji];
  const int tile = (int)(b - jb.b0);
  const int n = *jb.count, base = tile * TS_TILE;
  // no radix pass moves any digit of this list
  if (tile == 0 && threadIdx.x == 0) ds->sort_trivial[jb.id] = ~0u;
  if (base >= n) return;
  const int tn = min(TS_TILE, n - base);
  const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
  auto& s_key = lds.s_key;
  auto& s_val = lds.s_val;
  const int p0 = wv * (TS_ITEMS * WAVE) + lane;
  uint64_t key[TS_ITEMS];
  uint32_t val[TS_ITEMS];
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    const int q = base + min(p0 + j * WAVE, tn - 1);  // past the end: the last key again
    key[j] = jb.k[0][q];
    val[j] = jb.v[0][q];
  }
  // the tile's smallest and largest segment and time
  TileBits bits;
  bits.wb = jb.wb;
  bits.mask = (1ull << jb.wb) - 1;
  uint64_t ext[4] = {0, 0, 0, 0};  // largest ~segment, segment, ~time, time
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    const uint64_t sg = key[j] >> jb.wb, tm = key[j] & bits.mask;
    ext[0] = max(ext[0], ~sg);
    ext[1] = max(ext[1], sg);
    ext[2] = max(ext[2], ~tm);
    ext[3] = max(ext[3], tm);
  }
  tile_max(lds, ext);
  bits.seg0 = ~ext[0];
  bits.t0 = ~ext[2];
  bits.tb = bits_of(ext[3] - bits.t0);
  const int rb = bits_of(ext[1] - bits.seg0) + bits.tb;
  // Two passes order the tile by the top 16 of these bits: of 4096 keys few
  // share them, and those that do count their way past one
  // another.  (With every digit sorted the launch took 25 us on 60k rows,
  // against 21.)  Runs too long to count through take further passes: of keys
  // equal in the top bits, every digit from the lowest; of ops of equal key
  // (starts on a coarse clock), their end times first, then the digits again.
  // (60k rows with starts on a 30 ms grid: 138 us a call, 126 with starts as
  // they were; counting through runs of any length, each step a gather of two
  // end times, 940.)
  auto is_op = [&](uint64_t k) { return jb.contain && (k & 1) == 0; };
  auto end = [&](int j) { return (uint64_t)jobs.te[val[j]] ^ SIGN64; };
  int sh = rb > 16 ? rb - 16 : 0;  // bits not sorted
  bool ends = false, by_end = false;  // end times were sorted, are being sorted
  uint64_t last = 0;                  // the latest of the tile's ops
  for (int lo = sh, hi = rb;;) {
    for (int d = lo; d < hi; d += 8) {
      uint32_t dg[TS_ITEMS];
#pragma unroll
      for (int j = 0; j < TS_ITEMS; ++j) {
        // end times down; launches keep their order
        const uint64_t x = !by_end ? bits(key[j]) : is_op(key[j]) ? last - end(j) : 0;
        dg[j] = p0 + j * WAVE < tn ? (uint32_t)(x >> d) & 255u : 255u;
      }
      tile_pass(lds, ds, key, val, dg);
    }
    lo = 0;
    hi = rb;
    if (by_end) {
      by_end = false;
      continue;
    }
    tile_store(lds, key, val, p0);
    if (sh == 0 && (ends || !jb.contain)) break;
    bool far = false;
#pragma unroll
    for (int j = 0; j < TS_ITEMS; ++j) {
      const int p = p0 + j * WAVE + TS_RUN;
      if (p < tn) far |= (bits(s_key[p]) >> sh) == (bits(key[j]) >> sh) && (sh > 0 || is_op(key[j]));
    }
    if (!__syncthreads_or(far)) break;
    if (sh > 0) {
      sh = 0;
      continue;
    }
    uint64_t te[2] = {0, 0};  // largest ~end, end of an op
#pragma unroll
    for (int j = 0; j < TS_ITEMS; ++j) {
      if (p0 + j * WAVE >= tn || !is_op(key[j])) continue;
      te[0] = max(te[0], ~end(j));
      te[1] = max(te[1], end(j));
    }
    tile_max(lds, te);
    last = te[1];
    hi = bits_of(last - ~te[0]);
    ends = by_end = true;
  }
  if (sh == 0 && (ends || !jb.contain)) {  // what is equal is in row order
#pragma unroll
    for (int j = 0; j < TS_ITEMS; ++j) {
      const int p = p0 + j * WAVE;
      if (p >= tn) continue;
      jb.k[1][base + p] = key[j];
      jb.v[1][base + p] = val[j];
      if (p % TS_STEP == 0) jb.samples[tile * WAVE + p / TS_STEP] = key[j];
    }
    return;
  }
  // (a run of launches of equal key may be long: they keep their order)
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    const int p = p0 + j * WAVE;
    if (p >= tn) continue;
    const uint64_t k = key[j], h = bits(k) >> sh;
    const bool op = is_op(k), counts = sh > 0 || op;
    int to = p;
    for (int q = p - 1; counts && q >= 0; --q) {  // those before that belong after
      const uint64_t o = s_key[q];
      if ((bits(o) >> sh) != h) break;
      to -= o > k || (op && o == k && jobs.te[s_val[q]] < jobs.te[val[j]]);
    }
    for (int q = p + 1; counts && q < tn; ++q) {  // those after that belong before
      const uint64_t o = s_key[q];
      if ((bits(o) >> sh) != h) break;
      to += o < k || (op && o == k && jobs.te[s_val[q]] > jobs.te[val[j]]);
    }
    if (in_range(ds, to, tn)) {
      jb.k[1][base + to] = k;
      jb.v[1][base + to] = val[j];
    }
    if (to % TS_STEP == 0) jb.samples[tile * WAVE + to / TS_STEP] = k;
  }
}

struct TileMergeLds {
  uint64_t s_samp[TS_TILES][WAVE];
};

// One key per thread; TM_BATCH tiles are searched side by side, first their
// samples in LDS, then the TS_STEP keys after the last sample that counts,
// in memory (a wave's keys are neighbours, and so are the keys they read).
// Staging the stretch of every other tile that a chunk of keys spans instead
// took 20 us on a 60k-row window, but 60 where a long op, delivered at its
// end, sorts in front of its tile and stretches the first chunk.
constexpr int TM_BATCH = 8;
static_assert(TS_TILES % TM_BATCH == 0, "whole batches of tiles");

__device__ __forceinline__ void tile_merge_body(const TileSortJobs& jobs, DevState* ds, TileMergeLds& lds, uint32_t b) {
  int ji = 0;
  while (ji + 1 < jobs.m && b >= jobs.j[ji + 1].m0) ++ji;
  const TileSortJob& jb = jobs.j[ji];
  const int n = *jb.count;
  const int first = (int)(b - jb.m0) * TM_THREADS;
  if (first >= n) return;
  const int tile = first / TS_TILE, tiles = (n + TS_TILE - 1) / TS_TILE;
  const int tid = threadIdx.x, i = min(first + tid, n - 1);
  const uint64_t* ks = jb.k[1];
  const uint32_t* vs = jb.v[1];
  const uint64_t key = ks[i];
  const uint32_t val = vs[i];
  for (int x = tid; x < tiles * WAVE; x += TM_THREADS) {
    const int t = x / WAVE, ns = (min(TS_TILE, n - t * TS_TILE) + TS_STEP - 1) / TS_STEP;
    if (x % WAVE < ns) (&lds.s_samp[0][0])[x] = jb.samples[x];
  }
  __syncthreads();
  const bool op = jb.contain && (key & 1) == 0;
  int pos = i - tile * TS_TILE;
  // keys of equal value in an earlier tile come first (rows ascend from tile
  // to tile)
  for (int t0 = 0; t0 < tiles && tiles > 1; t0 += TM_BATCH) {  // uniform over the workgroup
    int len[TM_BATCH], q[TM_BATCH], w[TM_BATCH];
    auto counts = [&](int u, uint64_t x) { return t0 + u > tile ? x < key : x <= key; };
#pragma unroll
    for (int u = 0; u < TM_BATCH; ++u) {
      len[u] = t0 + u == tile ? 0 : max(0, min(TS_TILE, n - (t0 + u) * TS_TILE));
      w[u] = (len[u] + TS_STEP - 1) / TS_STEP;
      q[u] = 0;
    }
    for (int st = 0; st < 6; ++st) {  // the last sample that counts (or the first)
      uint64_t x[TM_BATCH];
#pragma unroll
      for (int u = 0; u < TM_BATCH; ++u) x[u] = lds.s_samp[t0 + u][q[u] + (w[u] >> 1)];
#pragma unroll
      for (int u = 0; u < TM_BATCH; ++u) {
        const int half = w[u] >> 1;
        q[u] = counts(u, x[u]) ? q[u] + half : q[u];
        w[u] -= half;
      }
    }
    bool some[TM_BATCH];
#pragma unroll
    for (int u = 0; u < TM_BATCH; ++u) {
      some[u] = len[u] > 0 && counts(u, lds.s_samp[t0 + u][q[u]]);
      q[u] = some[u] ? q[u] * TS_STEP : 0;
      w[u] = some[u] ? min(TS_STEP, len[u] - q[u]) : 0;  // the key at q counts
    }
    for (int st = 0; st < 6; ++st) {  // the last key that counts
      uint64_t x[TM_BATCH];
#pragma unroll
      for (int u = 0; u < TM_BATCH; ++u) x[u] = ks[min((t0 + u) * TS_TILE + q[u] + (w[u] >> 1), n - 1)];
#pragma unroll
      for (int u = 0; u < TM_BATCH; ++u) {
        const int half = w[u] >> 1;
        q[u] = half > 0 && counts(u, x[u]) ? q[u] + half : q[u];
        w[u] -= half;
      }
    }
#pragma unroll
    for (int u = 0; u < TM_BATCH; ++u) q[u] += some[u] ? 1 : 0;  // keys that count
    if (op) {
      // ops that start together: the run of equal keys (before q in an
      // earlier tile, from q on in a later one) is in end time order; those
      // that end later come first, in an earlier tile also those that end
      // as late
      uint64_t x[TM_BATCH];
#pragma unroll
      for (int u = 0; u < TM_BATCH; ++u)
        x[u] = ks[min((t0 + u) * TS_TILE + max(q[u] - (t0 + u > tile ? 0 : 1), 0), n - 1)];
#pragma unroll
      for (int u = 0; u < TM_BATCH; ++u) {
        const bool later = t0 + u > tile;
        if (len[u] == 0 || x[u] != key || (later ? q[u] >= len[u] : q[u] == 0)) continue;
        const int tb = (t0 + u) * TS_TILE;
        // the run's other end: steps doubled while the key is equal, then halved
        const int from = later ? q[u] : q[u] - 1, room = later ? len[u] - 1 - from : from, dir = later ? 1 : -1;
        int run = 0, step = 1;  // the key `run` steps on is equal
        while (run + step <= room && ks[tb + from + dir * (run + step)] == key) {
          run += step;
          step *= 2;
        }
        for (step >>= 1; step > 0; step >>= 1)
          if (run + step <= room && ks[tb + from + dir * (run + step)] == key) run += step;
        int a = later ? from : from - run, e = later ? from + run + 1 : q[u];
        const int64_t own = jobs.te[val];
        while (a < e) {
          const int mid = (a + e) >> 1;
          const int64_t o = jobs.te[vs[tb + mid]];
          if (later ? o > own : o >= own)
            a = mid + 1;
          else
            e = mid;
        }
        q[u] = a;
      }
    }
#pragma unroll
    for (int u = 0; u < TM_BATCH; ++u) pos += q[u];
  }
  if (first + tid < n && in_bounds(ds, pos, n)) {
    jb.k[0][pos] = key;
    jb.v[0][pos] = val;
  }
}

// Jobs of the lists that the call sorts; the grids of the two launches.
static inline TileSortJobs tile_sort_jobs(const Ctx& c, SortBufs* const* s, const int32_t* const* count, int k,
                                          int64_t* sort_grid, int64_t* merge_grid) {
  TileSortJobs jobs{};
  jobs.te = c.ev.te;
  int64_t b = 0, m = 0;
  const int64_t tiles = cdiv(std::min(std::max<int64_t>(c.n, 1), TS_ROWS), TS_TILE);
  uint64_t* samples = reinterpret_cast<uint64_t*>(c.hist_part);
  for (int i = 0; i < k; ++i) {
    jobs.j[jobs.m++] = TileSortJob{{s[i]->k[0], s[i]->k[1]}, {s[i]->v[0], s[i]->v[1]}, count[i],
                                   samples + (int64_t)s[i]->id * tiles * WAVE,
                                   s[i]->id == SORT_E ? c.wb1 : c.wb + (s[i]->id == SORT_C ? 1 : 0),
                                   s[i]->id == SORT_C ? 1 : 0,
                                   s[i]->id, (uint32_t)b, (uint32_t)m};
    b += tiles;
    m += tiles * (TS_TILE / TM_THREADS);
  }
  *sort_grid = b;
  *merge_grid = m;
  return jobs;
}

}  // namespace hx
