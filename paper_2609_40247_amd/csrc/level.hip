// Small windows: the call's kernels fused level by level.
//
// A small call is a chain of dependent kernels of a few microseconds each
// whatever their size, and 25 launches with 13 event operations on the host.
// Its three chains after the sorts (containment, join and names, timeline
// and overlap) need no streams of their own here: kernels that do not depend
// on each other run as slices of one launch on the caller's stream, so the
// chain is 13 launches long (nine for the smallest, whose lists are sorted in
// two launches instead of six), with no event and no second queue.  Each slice
// is a body that the full-size path launches by itself, over a range of the
// launch's workgroups; a workgroup has the threads of the widest body in the
// launch, and those that its own body does not use leave at once (a barrier
// counts only the waves still there).  LDS is sized per launch for the
// largest slice.
//
// A body's tiles wait only for tiles of lower index (look-backs), whose
// workgroups have lower indices here too.
#include "contain.hpp"
#include "crit.hpp"
#include "frame.hpp"
#include "graph.hpp"
#include "join.hpp"
#include "names.hpp"
#include "overlap.hpp"
#include "prep.hpp"
#include "radix.hpp"
#include "sol.hpp"
#include "tilesort.hpp"
#include "timeline.hpp"
#include "waits.hpp"

namespace hx {

enum : int {
  LJ_INIT, LJ_PREP, LJ_TABLE, LJ_TSORT, LJ_TMERGE, LJ_HIST, LJ_PLAN, LJ_PASS, LJ_REFINE, LJ_STORE, LJ_RESOLVE, LJ_DUPS, LJ_FIX, LJ_EDGES, LJ_NAMES,
  LJ_NAMES_FOLD, LJ_OPNAMES, LJ_OPNAMES_FOLD, LJ_KERNEL_OPS, LJ_UNION, LJ_UNION_D, LJ_UNION_O, LJ_SEGOFF, LJ_SWEEP,
  LJ_SWEEP_MANY, LJ_VBUILD, LJ_QUERY, LJ_DEPTH, LJ_OPAGG, LJ_NOCONTAIN,
  LJ_DG_SCAN, LJ_WAITS, LJ_GRAPH, LJ_GRAPH_FOLD, LJ_SOL, LJ_SOL_FOLD, LJ_SOL_NAMES, LJ_CRIT_KERNELS, LJ_CRIT_HOST,
  LJ_CRIT_LAST, LJ_CRIT_OPS, LJ_CRIT_ROWS, LJ_CRIT_LOCAL
};
constexpr int LV_SLICES = 8;

struct LevelSlice {
  int job;
  uint32_t b0;      // the slice's first workgroup
  uint32_t gx, gy;  // its grid
};
struct LevelArgs {
  LevelSlice s[LV_SLICES];
  int n;
  bool packed;  // the sorts move packed words
  DevState* ds;
  union {
    struct {  // up to the sorted lists
      InitArgs init;
      PrepArgs prep;
      HistJobs hist;
      union {  // one of them per launch
        TileSortJobs tsort;
        SortJobs sort;
        RefineJobs refine;
      };
    };
    struct {  // after them: the optional outputs
      WaitsArgs waits;
      GraphArgs graph;
      SolArgs sol;
      CritArgs crit;
      int sol_blocks;
    };
  };
  JoinArgs join;
  NamesArgs names;
  OpNamesArgs opnames;
  UnionArgs uni;
  UnionArgs uni_d;
  UnionArgs uni_o;
  SweepArgs sweep;
  ContainArgs con;
};
static_assert(sizeof(LevelArgs) <= 4096, "kernel arguments");

template <class T>
__device__ __forceinline__ T& level_lds_as(char* p) {
  return *reinterpret_cast<T*>(p);
}

constexpr int LV_THREADS = 1024;

// The arguments are read where the launch put them: a copy of the struct in
// private memory (what passing parts of it on by reference makes of a kernel
// parameter this large) took 65 us a launch.
__global__ __launch_bounds__(LV_THREADS) void k_level(LevelArgs) {
  extern __shared__ __align__(16) char lds[];
  const LevelArgs& a = *(const LevelArgs*)(const void*)__builtin_amdgcn_kernarg_segment_ptr();
  int i = 0;
  while (i + 1 < a.n && blockIdx.x >= a.s[i + 1].b0) ++i;
  const LevelSlice sl = a.s[i];
  const uint32_t b = blockIdx.x - sl.b0, gx = sl.gx, gy = sl.gy;
  const uint32_t by = gy > 1 ? b / gx : 0u, bx = gy > 1 ? b - by * gx : b;
  const int t = threadIdx.x;
  switch (sl.job) {
    case LJ_INIT:
      if (t < 256) init_body(a.init, bx, gx);
      break;
    case LJ_PREP:
      if (t < PREP_THREADS) prep_body<PREP_ITEMS_SMALL>(a.prep, level_lds_as<PrepLds<PREP_ITEMS_SMALL>>(lds), bx);
      break;
    case LJ_TABLE:
      if (t < HIST_THREADS) jt_empty_body(a.hist, a.ds, level_lds_as<JtEmptyLds>(lds), bx, gx);
      break;
    case LJ_TSORT:
      if (t < TS_THREADS) tile_sort_body(a.tsort, a.ds, level_lds_as<TileSortLds>(lds), bx);
      break;
    case LJ_TMERGE:
      if (t < TM_THREADS) tile_merge_body(a.tsort, a.ds, level_lds_as<TileMergeLds>(lds), bx);
      break;
    case LJ_HIST:
      if (t < HIST_THREADS) digit_hist_body(a.hist, a.ds, level_lds_as<DigitHistLds>(lds), bx, by, gx);
      break;
    case LJ_PLAN:
      if (t < PLAN_THREADS) hist_plan_body(a.hist, a.ds, level_lds_as<HistPlanLds>(lds), bx, by);
      break;
    case LJ_PASS:
      if (t >= RS_THREADS) break;
      if (a.packed)
        radix_pass_body<true>(a.sort, a.ds, level_lds_as<RadixPassLds<true>>(lds), bx);
      else
        radix_pass_body<false>(a.sort, a.ds, level_lds_as<RadixPassLds<false>>(lds), bx);
      break;
    case LJ_REFINE:
      if (t >= RF_THREADS) break;
      if (a.packed)
        refine_body<true>(a.refine, a.ds, level_lds_as<RefineLds>(lds), bx, by);
      else
        refine_body<false>(a.refine, a.ds, level_lds_as<RefineLds>(lds), bx, by);
      break;
    case LJ_STORE:
      if (t < 256) jt_store_body<1>(a.join, bx);
      break;
    case LJ_RESOLVE:
      if (t < 256) jt_resolve_body<1>(a.join, level_lds_as<JtResolveLds>(lds), bx);
      break;
    case LJ_DUPS:
      if (t < 256) jt_dups_body(a.join, bx, gx);
      break;
    case LJ_FIX:
      if (t < 256) jt_fix_body(a.join, level_lds_as<JtFixLds>(lds), bx, gx);
      break;
    case LJ_EDGES:
      if (t < 256) edges_body(a.join, bx, gx);
      break;
    case LJ_NAMES:
      if (t < NM_THREADS) names_partial_body(a.names, reinterpret_cast<unsigned long long*>(lds), bx, gx);
      break;
    case LJ_NAMES_FOLD:
      if (t < 256) names_reduce_body(a.names, bx, by);
      break;
    case LJ_OPNAMES:
      if (t < ON_THREADS) opnames_partial_body(a.opnames, reinterpret_cast<unsigned long long*>(lds), bx, gx);
      break;
    case LJ_OPNAMES_FOLD:
      if (t < 256) opnames_fold_body(a.opnames, bx, by, gy);
      break;
    case LJ_KERNEL_OPS:
      if (t < KO_THREADS) kernel_ops_body(a.names, bx);
      break;
    case LJ_UNION:
      if (t < UN_THREADS_SMALL) union_body<UN_THREADS_SMALL>(a.uni, level_lds_as<UnionLds<UN_THREADS_SMALL>>(lds), bx);
      break;
    case LJ_UNION_D:
      if (t < UN_THREADS_SMALL) union_body<UN_THREADS_SMALL>(a.uni_d, level_lds_as<UnionLds<UN_THREADS_SMALL>>(lds), bx);
      break;
    case LJ_UNION_O:
      if (t < UN_THREADS_SMALL) union_body<UN_THREADS_SMALL>(a.uni_o, level_lds_as<UnionLds<UN_THREADS_SMALL>>(lds), bx);
      break;
    case LJ_SEGOFF:
      if (t < 256) segoff_body(a.sweep, bx, gx);
      break;
    case LJ_SWEEP:
      if (t < SW_THREADS) sweep_groups_body<SW_ITEMS_SMALL>(a.sweep, level_lds_as<SweepGroupsLds>(lds), bx);
      break;
    case LJ_SWEEP_MANY:
      if (t < SM_THREADS)
        sweep_many_body(a.sweep, level_lds_as<SweepManyLds>(lds),
                        reinterpret_cast<unsigned long long*>(lds + sizeof(SweepManyLds)), bx, gx);
      break;
    case LJ_VBUILD:
      if (t < VB_THREADS) vbuild_body(a.con, level_lds_as<VbuildLds>(lds), bx);
      break;
    case LJ_QUERY:
      if (t < QY_THREADS) query_body(a.con, level_lds_as<QueryLds>(lds), bx);
      break;
    case LJ_DEPTH:
      if (t < 256) depth_body(a.con, level_lds_as<DepthLds>(lds), bx);
      break;
    case LJ_OPAGG:
      if (t < AG_THREADS) opagg_body(a.con, level_lds_as<OpaggLds>(lds), bx);
      break;
    case LJ_NOCONTAIN:
      if (t < 256) nocontain_body(a.con.k[0], a.con.v[0], a.ds, a.con.link, a.con.aux, bx, gx);
      break;
    case LJ_DG_SCAN:
      if (t < DG_THREADS) dg_scan_body(a.waits, level_lds_as<DgScanLds>(lds), bx);
      break;
    case LJ_WAITS:
      if (t < WT_THREADS) waits_body(a.waits, level_lds_as<WaitsLds>(lds), bx, gx);
      break;
    case LJ_GRAPH:
      if (t < GR_THREADS) graph_body(a.graph, reinterpret_cast<unsigned long long*>(lds), bx, gx);
      break;
    case LJ_GRAPH_FOLD:
      if (t < 256) graph_fold_body(a.graph, bx, by, gy);
      break;
    case LJ_SOL:
      if (t < SOL_THREADS) sol_body(a.sol, reinterpret_cast<unsigned long long*>(lds), bx, gx);
      break;
    case LJ_SOL_FOLD:
      if (t < 256) sol_fold_body(a.sol, a.sol_blocks, bx, by, gy);
      break;
    case LJ_SOL_NAMES:
      if (t < 256) sol_names_body(a.sol, bx);
      break;
    case LJ_CRIT_KERNELS:
      if (t < 256) crit_kernels_body(a.crit, level_lds_as<CritKernelsLds>(lds), bx, gx);
      break;
    case LJ_CRIT_HOST:
      if (t < 256) crit_host_body(a.crit, level_lds_as<CritHostLds>(lds), bx, gx);
      break;
    case LJ_CRIT_LAST:
      if (t < 256) crit_last_body(a.crit, bx, gx);
      break;
    case LJ_CRIT_OPS:
      if (t < 256) crit_ops_body(a.crit, bx, gx);
      break;
    case LJ_CRIT_ROWS:
      if (t < 256) crit_rows_body(a.crit, bx, gx);
      break;
    default:  // LJ_CRIT_LOCAL
      if (t < CP_LT) crit_local_body(a.crit, level_lds_as<CritLocalLds>(lds), bx);
      break;
  }
}

static_assert(sizeof(SweepManyLds) % 8 == 0, "the pair sums follow it");

// Collects slices and launches them as one grid.
struct Level {
  Ctx& c;
  LevelArgs& a;
  uint32_t blocks = 0;
  int threads = 64;
  size_t lds = 0;
  Level(Ctx& c_, LevelArgs& a_) : c(c_), a(a_) {}
  void add(int job, int64_t gx, int64_t gy, int th, size_t bytes) {
    if (gx <= 0 || gy <= 0) return;
    a.s[a.n++] = LevelSlice{job, blocks, (uint32_t)gx, (uint32_t)gy};
    blocks += (uint32_t)(gx * gy);
    threads = std::max(threads, th);
    lds = std::max(lds, bytes);
  }
  void launch() {
    if (a.n == 0) return;
    hipLaunchKernelGGL(k_level, dim3(blocks), dim3((unsigned)threads), lds, c.st, a);
    a.n = 0;
    blocks = 0;
    threads = 64;
    lds = 0;
  }
};

// The whole call up to the critical path's walk; that and the last kernel
// follow on the same stream.
void launch_levels(Ctx& c, SortBufs* const* ss, const int32_t* const* cc, int ks, int passes) {
  LevelArgs a{};
  a.ds = c.ds;
  a.packed = c.packed;
  a.init = init_args(c);
  a.prep = prep_args(c);
  int64_t hist_grid;
  int hist_m, hist_nd;
  a.hist = hist_jobs(c, ss, cc, ks, &hist_grid, &hist_m, &hist_nd);
  a.join = join_args(c);
  a.names = names_args(c);
  a.opnames = opnames_args(c);
  a.uni = timeline_args(c);
  if (c.waits) {
    a.uni_d = union_device_args(c);
    a.uni_o = union_opnames_args(c);
  }
  a.sweep = sweep_args(c);
  a.con = contain_args(c);
  const bool rows = c.n > 0, names = names_wanted(c), fold = names && c.NN <= NM_LDS_NAMES, opn = opnames_wanted(c);
  const int64_t ct = std::max<int64_t>(cdiv(c.sC.n_max, CT_TILE), 1);
  Level l(c, a);
  // The join's steps, one a launch from the emptied table on (its list is
  // prep's): the last before the per-op aggregates
  int step = 0;
  auto join_step = [&]() {
    if (!rows) return;
    switch (step++) {
      case 0: l.add(LJ_STORE, jt_blocks(c, 1), 1, 256, 0); break;
      case 1: l.add(LJ_RESOLVE, jt_blocks(c, 1), 1, 256, sizeof(JtResolveLds)); break;
      case 2: l.add(LJ_DUPS, jt_fix_blocks(c), 1, 256, 0); break;
      case 3: l.add(LJ_FIX, jt_fix_blocks(c), 1, 256, sizeof(JtFixLds)); break;
      default: break;
    }
  };

  l.add(LJ_INIT, init_blocks(c, a.init), 1, 256, 0);
  l.launch();
  if (rows) {
    l.add(LJ_PREP, c.prep_tiles, 1, PREP_THREADS, sizeof(PrepLds<PREP_ITEMS_SMALL>));
    l.launch();
    if (c.crit) launch_crit_elist(c);
  }
  // the sorts, the names' tables and the first steps of the join
  const size_t names_lds = c.NN <= NM_LDS_NAMES ? (size_t)c.NN * 32 : 0;
  auto tables = [&]() {
    if (names) l.add(LJ_NAMES, c.name_blocks, 1, NM_THREADS, names_lds);
    if (opn && rows) l.add(LJ_OPNAMES, c.opn_blocks, 1, ON_THREADS, a.opnames.lds ? (size_t)c.NOP * 32 : 0);
  };
  auto names_fold = [&]() {
    if (opn && rows && a.opnames.lds)
      l.add(LJ_OPNAMES_FOLD, cdiv((int64_t)c.NOP * 4, 256), opnames_fold_rows(c), 256, 0);
    if (fold) l.add(LJ_NAMES_FOLD, cdiv((int64_t)c.NN * 4, 256), names_fold_rows(c), 256, 0);
  };
  if (c.n <= TS_ROWS) {
    int64_t sort_grid, merge_grid;
    a.tsort = tile_sort_jobs(c, ss, cc, ks, &sort_grid, &merge_grid);
    l.add(LJ_TSORT, sort_grid, 1, TS_THREADS, sizeof(TileSortLds));
    l.add(LJ_TABLE, std::min<int64_t>(cdiv(2 * std::max<int64_t>(c.n, 1), HIST_CHUNK), HIST_MAX_BLOCKS), 1,
          HIST_THREADS, sizeof(JtEmptyLds));
    tables();
    l.launch();
    l.add(LJ_TMERGE, merge_grid, 1, TM_THREADS, sizeof(TileMergeLds));
    join_step();
    names_fold();
    l.launch();
  } else {
    l.add(LJ_HIST, hist_grid, hist_m + 1, HIST_THREADS, sizeof(DigitHistLds));
    tables();
    l.launch();
    l.add(LJ_PLAN, hist_nd, hist_m, PLAN_THREADS, sizeof(HistPlanLds));
    join_step();
    names_fold();
    l.launch();
    for (int p = 0; p < passes; ++p) {
      int64_t grid;
      a.sort = sort_jobs(c, ss, cc, ks, p, &grid);
      if (a.sort.m > 0)
        l.add(LJ_PASS, grid, 1, RS_THREADS, c.packed ? sizeof(RadixPassLds<true>) : sizeof(RadixPassLds<false>));
      join_step();
      l.launch();
    }
    int64_t grid;
    int m;
    a.refine = refine_jobs(c, &grid, &m);
    if (m > 0) l.add(LJ_REFINE, grid, m, RF_THREADS, sizeof(RefineLds));
    join_step();
    l.launch();
  }

  // the sorted lists are there
  if (c.waits) a.waits = waits_args(c);
  if (c.graph) a.graph = graph_args(c);
  if (c.sol) {
    a.sol = sol_args(c);
    a.sol_blocks = c.sol_blocks;
  }
  if (c.crit) a.crit = crit_args(c);
  l.add(LJ_UNION, c.union_tiles, 1, UN_THREADS_SMALL, sizeof(UnionLds<UN_THREADS_SMALL>));
  if (c.contain) l.add(LJ_VBUILD, ct, 1, VB_THREADS, sizeof(VbuildLds));
  if (c.waits) {
    l.add(LJ_UNION_D, c.union_tiles, 1, UN_THREADS_SMALL, sizeof(UnionLds<UN_THREADS_SMALL>));
    l.add(LJ_UNION_O, c.union_tiles, 1, UN_THREADS_SMALL, sizeof(UnionLds<UN_THREADS_SMALL>));
  }
  join_step();
  if (!c.contain && (c.o.link || c.o.aux))
    l.add(LJ_NOCONTAIN, std::min<int64_t>(std::max<int64_t>(cdiv(c.n, 256 * 8), 1), 2048), 1, 256, 0);
  l.launch();

  if (c.contain) l.add(LJ_QUERY, ct, 1, QY_THREADS, sizeof(QueryLds));
  if (c.overlap) l.add(LJ_SEGOFF, segoff_blocks(c), 1, 256, 0);
  join_step();
  if (c.waits) l.add(LJ_DG_SCAN, c.dg_tiles, 1, DG_THREADS, sizeof(DgScanLds));
  l.launch();

  if (c.overlap) {
    if (sweep_by_groups(c))
      l.add(LJ_SWEEP, sweep_groups_blocks(c, SW_ITEMS_SMALL), 1, SW_THREADS, sizeof(SweepGroupsLds));
    else
      l.add(LJ_SWEEP_MANY, sweep_many_blocks(c), 1, SM_THREADS, sizeof(SweepManyLds) + (size_t)c.S * c.S * 8);
  }
  if (c.contain) l.add(LJ_DEPTH, std::max<int64_t>(cdiv(c.sC.n_max, 256 * DP_ITEMS), 1), 1, 256, sizeof(DepthLds));
  join_step();
  if (c.waits) l.add(LJ_WAITS, waits_blocks(c), 1, WT_THREADS, sizeof(WaitsLds));
  l.launch();

  if (c.contain) {
    l.add(LJ_OPAGG, std::max<int64_t>(cdiv(c.sC.n_max, AG_TILE), 1), 1, AG_THREADS, sizeof(OpaggLds));
    l.add(LJ_KERNEL_OPS, kernel_ops_blocks(c), 1, KO_THREADS, 0);
  }
  if (c.p.n_edges > 0) l.add(LJ_EDGES, std::min<int64_t>(cdiv(c.p.n_edges, 256), 1024), 1, 256, 0);
  const int64_t cg = crit_grid(c.n);
  if (c.crit && rows) {
    l.add(LJ_CRIT_HOST, cg, 1, 256, sizeof(CritHostLds));
    l.add(LJ_CRIT_KERNELS, cg, 1, 256, sizeof(CritKernelsLds));
  }
  if (c.graph) l.add(LJ_GRAPH, c.graph_blocks, 1, GR_THREADS, a.graph.lds ? (size_t)c.NG * GR_STATS * 8 : 0);
  l.launch();

  if (c.sol) l.add(LJ_SOL, c.sol_blocks, 1, SOL_THREADS, a.sol.lds ? (size_t)c.NOP * 32 : 0);
  if (c.crit && rows) l.add(LJ_CRIT_LAST, cg, 1, 256, 0);
  if (c.graph && a.graph.lds)
    l.add(LJ_GRAPH_FOLD, cdiv((int64_t)c.NG * GR_STATS, 256), graph_fold_rows(c), 256, 0);
  l.launch();

  if (c.sol && a.sol.lds)
    l.add(LJ_SOL_FOLD, cdiv((int64_t)c.NOP * 4, 256), std::min(SF_ROWS, c.sol_blocks), 256, 0);
  if (c.crit && rows) {
    l.add(LJ_CRIT_OPS, cg, 1, 256, 0);
    l.add(LJ_CRIT_ROWS, cg, 1, 256, 0);
  }
  l.launch();

  if (c.sol) l.add(LJ_SOL_NAMES, cdiv(c.NOP, 256), 1, 256, 0);
  if (c.crit && rows) l.add(LJ_CRIT_LOCAL, cdiv(2 * c.n, CP_TE), 1, CP_LT, sizeof(CritLocalLds));
  l.launch();
}

hipError_t level_set_lds_attr() {
  return hipFuncSetAttribute((const void*)k_level, hipFuncAttributeMaxDynamicSharedMemorySize, NM_LDS_NAMES * 32);
}

}  // namespace hx
