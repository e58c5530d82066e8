// Sort of the lists of a small window in two launches, in place of the digit
// histogram, its plan, the radix passes and the refine pass (six launches
// whose few tiles leave most of the chip idle, about 50 us of the 140 of a
// 60k-row window).
//
//   tile sort: a workgroup sorts TS_TILE keys of a list in LDS (two passes of
//              the radix passes' ranking over the top bits of the keys'
//              range, then runs of equal bits by counting), and writes the
//              tile and every TS_STEP-th key of it;
//   merge:     a workgroup takes TS_CHUNK consecutive keys of a sorted tile
//              and finds, for every other tile, how many of its keys come
//              before each of them: the sampled keys bound the stretch of
//              the tile that can matter, which is staged in LDS and searched.
//              The sum is the key's place.
//
// In a trace in delivery order a chunk's keys fall among those of a few tiles
// only; in no order among all of them, and the merge costs a search per key
// and tile, which is what bounds the number of tiles (TS_TILES).
#pragma once

#include "internal.hpp"

namespace hx {

constexpr int TS_THREADS = 1024;
constexpr int TS_ITEMS = TS_TILE / TS_THREADS;
constexpr int TS_WAVES = TS_THREADS / WAVE;
constexpr int TS_STEP = TS_TILE / WAVE;  // keys between samples: a wave's lanes hold a tile's samples
static_assert(TS_ITEMS * TS_THREADS == TS_TILE && TS_THREADS >= 256, "one thread per digit value");
constexpr int TM_THREADS = 256;
constexpr int TM_ITEMS = 2;
constexpr int TS_CHUNK = TM_THREADS * TM_ITEMS;
static_assert(TS_TILE % TS_CHUNK == 0, "chunks divide a tile");

struct TileSortJob {
  uint64_t* k[2];  // prep's list, and the result; the sorted tiles
  uint32_t* v[2];
  const int32_t* count;
  uint64_t* samples;  // [TS_TILES][WAVE]
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
  uint64_t s_min[TS_WAVES], s_max[TS_WAVES];
};

// One stable pass over the tile by 8 bits of (key - lo) >> sh.  Item j of
// lane l is the tile's position (wave * TS_ITEMS + j) * 64 + l: items in
// order, lanes in order is the tile's order.  Positions from tn on stay last.
__device__ __forceinline__ void tile_pass(TileSortLds& lds, DevState* ds, uint64_t (&key)[TS_ITEMS],
                                          uint32_t (&val)[TS_ITEMS], uint64_t lo, int sh, int tn) {
  const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int p0 = wv * (TS_ITEMS * WAVE) + lane;
  auto& s_wh = lds.s_wh;
  constexpr int OR_XOR = 0xF0 | (0xCC ^ 0xAA);  // truth table of a | (b ^ c)
  for (int i = tid; i < TS_WAVES * 256; i += TS_THREADS) (&s_wh[0][0])[i] = 0;
  __syncthreads();
  uint32_t rank[TS_ITEMS], dg[TS_ITEMS];
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    dg[j] = p0 + j * WAVE < tn ? (uint32_t)((key[j] - lo) >> sh) & 255u : 255u;
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

constexpr int TS_RUN = 32;  // longest run of keys equal in the passes' bits that is ordered by counting

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
  // the tile's smallest and largest key
  uint64_t mn = key[0], mx = key[0];
#pragma unroll
  for (int j = 1; j < TS_ITEMS; ++j) {
    mn = key[j] < mn ? key[j] : mn;
    mx = key[j] > mx ? key[j] : mx;
  }
  mn = ~wave_allmax_u64(~mn);
  mx = wave_allmax_u64(mx);
  if (lane == 0) {
    lds.s_min[wv] = mn;
    lds.s_max[wv] = mx;
  }
  __syncthreads();
  mn = ~wave_allmax_u64(~(lane < TS_WAVES ? lds.s_min[lane] : ~0ull));
  mx = wave_allmax_u64(lane < TS_WAVES ? lds.s_max[lane] : 0ull);
  // Two passes order the tile by the top 16 bits of the keys' range: with
  // 4096 keys, few share them, and those that do count their way past one
  // another.  (Sorting every digit took five passes of about 3 us.)
  const int rb = bits_of(mx - mn);
  int sh = rb > 16 ? rb - 16 : 0;
  if (rb > 0) tile_pass(lds, ds, key, val, mn, sh, tn);
  if (rb > 8) tile_pass(lds, ds, key, val, mn, sh + 8, tn);
  __syncthreads();  // (the passes' reads of the tile)
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    s_key[p0 + j * WAVE] = key[j];
    s_val[p0 + j * WAVE] = val[j];
  }
  __syncthreads();
  if (sh > 0) {
    // a run too long to count through: every digit, from the lowest
    bool far = false;
#pragma unroll
    for (int j = 0; j < TS_ITEMS; ++j) {
      const int p = p0 + j * WAVE + TS_RUN;
      if (p < tn) far |= ((s_key[p] - mn) >> sh) == ((key[j] - mn) >> sh);
    }
    if (__syncthreads_or(far)) {
      for (int d = 0; d < rb; d += 8) tile_pass(lds, ds, key, val, mn, d, tn);
      sh = 0;
      __syncthreads();
#pragma unroll
      for (int j = 0; j < TS_ITEMS; ++j) {
        s_key[p0 + j * WAVE] = key[j];
        s_val[p0 + j * WAVE] = val[j];
      }
      __syncthreads();
    }
  }
#pragma unroll
  for (int j = 0; j < TS_ITEMS; ++j) {
    const int p = p0 + j * WAVE;
    if (p >= tn) continue;
    const uint64_t k = key[j], h = (k - mn) >> sh;
    const bool op = jb.contain && (k & 1) == 0;
    int to = p;
    for (int q = p - 1; q >= 0; --q) {  // those before that belong after
      const uint64_t o = s_key[q];
      if (((o - mn) >> sh) != h) break;
      to -= o > k || (op && o == k && jobs.te[s_val[q]] < jobs.te[val[j]]);
    }
    for (int q = p + 1; q < tn; ++q) {  // those after that belong before
      const uint64_t o = s_key[q];
      if (((o - mn) >> sh) != h) break;
      to += o < k || (op && o == k && jobs.te[s_val[q]] > jobs.te[val[j]]);
    }
    if (in_range(ds, to, tn)) {
      jb.k[1][base + to] = k;
      jb.v[1][base + to] = val[j];
    }
    if (to % TS_STEP == 0) jb.samples[tile * WAVE + to / TS_STEP] = k;
  }
}

constexpr int TM_GRAN = 64;  // granules (TS_STEP keys) staged at a time

struct TileMergeLds {
  uint64_t s_key[TM_GRAN * TS_STEP];
  uint32_t s_src[TM_GRAN];     // each staged granule's position in the list
  uint32_t s_lo[TS_TILES];     // per tile: the first position that can matter,
  uint32_t s_cnt[TS_TILES];    // keys from there on that can,
  uint32_t s_off[TS_TILES];    // granules before them, over the tiles
  uint64_t s_scan[TM_THREADS / WAVE];
};

__device__ __forceinline__ void tile_merge_body(const TileSortJobs& jobs, DevState* ds, TileMergeLds& lds, uint32_t b) {
  int ji = 0;
  while (ji + 1 < jobs.m && b >= jobs.j[ji + 1].m0) ++ji;
  const TileSortJob& jb = jobs.j[ji];
  const int n = *jb.count;
  const int first = (int)(b - jb.m0) * TS_CHUNK;  // the chunk's first position
  if (first >= n) return;
  const int tile = first / TS_TILE, tiles = (n + TS_TILE - 1) / TS_TILE;
  const int cn = min(TS_CHUNK, min(n, (tile + 1) * TS_TILE) - first);
  const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
  constexpr int NW = TM_THREADS / WAVE;
  auto& s_key = lds.s_key;
  const uint64_t* ks = jb.k[1];
  const uint32_t* vs = jb.v[1];
  uint64_t key[TM_ITEMS];
  uint32_t val[TM_ITEMS];
  int pos[TM_ITEMS];
#pragma unroll
  for (int j = 0; j < TM_ITEMS; ++j) {
    const int i = min(tid + j * TM_THREADS, cn - 1);
    key[j] = ks[first + i];
    val[j] = vs[first + i];
    pos[j] = first - tile * TS_TILE + i;
  }
  const uint64_t kf = ks[first], kl = ks[first + cn - 1];
  // Per other tile, from its samples (a lane each): the positions before lo
  // hold keys below every key of the chunk, those from lo + cnt on above.
  constexpr int TB = 8;  // tiles whose samples are in flight together
  for (int t0 = wv; t0 < tiles; t0 += TB * NW) {
    uint64_t s[TB];
#pragma unroll
    for (int u = 0; u < TB; ++u) {
      const int t = min(t0 + u * NW, tiles - 1);
      const int ns = (min(TS_TILE, n - t * TS_TILE) + TS_STEP - 1) / TS_STEP;
      s[u] = jb.samples[t * WAVE + min(lane, ns - 1)];
    }
#pragma unroll
    for (int u = 0; u < TB; ++u) {
      const int t = t0 + u * NW;
      if (t >= tiles) continue;  // uniform over the wave
      const int len = min(TS_TILE, n - t * TS_TILE), ns = (len + TS_STEP - 1) / TS_STEP;
      const int below = popc(ballot(lane < ns && s[u] < kf)), upto = popc(ballot(lane < ns && s[u] <= kl));
      const int lo = max(below - 1, 0) * TS_STEP, hi = min(upto * TS_STEP, len);
      if (lane == 0) {
        lds.s_lo[t] = t == tile ? 0u : (uint32_t)lo;
        lds.s_cnt[t] = t == tile ? 0u : (uint32_t)max(hi - lo, 0);
      }
    }
  }
  __syncthreads();
  static_assert(TS_TILES <= TM_THREADS, "one thread per tile");
  const uint32_t ng_t = tid < tiles ? (lds.s_cnt[tid] + TS_STEP - 1) / TS_STEP : 0u;
  const uint32_t lo_t = tid < tiles ? lds.s_lo[tid] : 0u;
  // granules before each tile's, and the keys before all the stretches
  uint64_t tot;
  const uint64_t ex = block_excl_sum<TM_THREADS>(((uint64_t)lo_t << 32) | ng_t, lds.s_scan, &tot);
  if (tid < tiles) lds.s_off[tid] = (uint32_t)ex;
  const int ng = (int)(uint32_t)tot;
#pragma unroll
  for (int j = 0; j < TM_ITEMS; ++j) pos[j] += (int)(tot >> 32);
  // The stretches' granules, TM_GRAN at a time, in LDS; a tile's part of
  // them is one sorted segment.
  for (int g0 = 0; g0 < ng; g0 += TM_GRAN) {  // uniform over the workgroup
    const int g1 = min(ng, g0 + TM_GRAN);
    __syncthreads();  // the offsets, and the last granules' reads
    for (int q = (int)(uint32_t)ex; q < (int)((uint32_t)ex + ng_t); ++q)
      if (q >= g0 && q < g1) lds.s_src[q - g0] = (uint32_t)(tid * TS_TILE) + lo_t + (uint32_t)(q - (int)(uint32_t)ex) * TS_STEP;
    __syncthreads();
    constexpr int GB = TM_GRAN / NW;  // granules per wave
    uint64_t v[GB];
#pragma unroll
    for (int u = 0; u < GB; ++u) {
      const int g = g0 + min(wv + u * NW, g1 - g0 - 1);
      v[u] = ks[min((int)lds.s_src[g - g0] + lane, n - 1)];
    }
#pragma unroll
    for (int u = 0; u < GB; ++u) s_key[(wv + u * NW) * TS_STEP + lane] = v[u];
    __syncthreads();
    for (int t = 0; t < tiles; ++t) {  // uniform over the workgroup
      const int off = (int)lds.s_off[t], cnt_t = (int)lds.s_cnt[t];
      const int ga = max(off, g0), gb = min(off + (cnt_t + TS_STEP - 1) / TS_STEP, g1);
      if (ga >= gb) continue;
      const uint64_t* seg = s_key + (ga - g0) * TS_STEP;
      const int seg0 = (ga - off) * TS_STEP;                 // the segment's first key in the stretch
      const int cnt = min((gb - off) * TS_STEP, cnt_t) - seg0;
      // keys of equal value in an earlier tile come first (rows ascend from
      // tile to tile)
      const bool later = t > tile;
      auto counts = [&](uint64_t x, uint64_t k) { return later ? x < k : x <= k; };
      int q[TM_ITEMS];
#pragma unroll
      for (int j = 0; j < TM_ITEMS; ++j) q[j] = 0;
      for (int w = cnt; w > 1;) {
        const int half = w >> 1;
        uint64_t x[TM_ITEMS];
#pragma unroll
        for (int j = 0; j < TM_ITEMS; ++j) x[j] = seg[q[j] + half];
#pragma unroll
        for (int j = 0; j < TM_ITEMS; ++j) q[j] = counts(x[j], key[j]) ? q[j] + half : q[j];
        w -= half;
      }
#pragma unroll
      for (int j = 0; j < TM_ITEMS; ++j) {
        int r = q[j] + (counts(seg[q[j]], key[j]) ? 1 : 0);  // keys that count
        if (jb.contain && (key[j] & 1) == 0) {
          // ops that start together: the segment's run of equal keys (before
          // r in an earlier tile, from r on in a later one) is in end time
          // order; those that end later come first, in an earlier tile also
          // those that end as late
          int a = r, e = r;
          if (later)
            while (e < cnt && seg[e] == key[j]) ++e;
          else
            while (a > 0 && seg[a - 1] == key[j]) --a;
          if (a < e) {
            const int64_t own = jobs.te[val[j]];
            const uint32_t* sv = vs + t * TS_TILE + (int)lds.s_lo[t] + seg0;
            int y = e;
            while (a < y) {
              const int mid = (a + y) >> 1;
              const int64_t o = jobs.te[sv[mid]];
              if (later ? o > own : o >= own)
                a = mid + 1;
              else
                y = mid;
            }
            r = a;
          }
        }
        pos[j] += r;
      }
    }
  }
#pragma unroll
  for (int j = 0; j < TM_ITEMS; ++j) {
    if (tid + j * TM_THREADS >= cn) continue;
    if (in_bounds(ds, pos[j], n)) {
      jb.k[0][pos[j]] = key[j];
      jb.v[0][pos[j]] = val[j];
    }
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
                                   samples + (int64_t)s[i]->id * tiles * WAVE, s[i]->id == SORT_C ? 1 : 0,
                                   s[i]->id, (uint32_t)b, (uint32_t)m};
    b += tiles;
    m += tiles * (TS_TILE / TS_CHUNK);
  }
  *sort_grid = b;
  *merge_grid = m;
  return jobs;
}

}  // namespace hx
