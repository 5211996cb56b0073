// mlproj: several independent bi-level projections in one chain of launches.
#ifndef MLPROJ_BATCH_H
#define MLPROJ_BATCH_H

#include "aggregate.h"
#include "common.h"
#include "l11.h"
#include "l11held.h"
#include "map.h"
#include "tiny.h"

namespace mlproj {

// A training loop projects many weight matrices after every step (the use Sec. 6.3 makes of
// the projection), most of them small enough that the three launches of a call are what it
// costs.  Up to BATCH_MAX matrices share one aggregate, one fold and one map launch (and,
// for l1,1, one launch per kernel of the inner searches): the
// problems travel in the kernel arguments, a workgroup finds the problem its number falls
// into and then runs exactly the code of the single-matrix kernels on it, with the geometry
// and workspace layout recomputed on the device from (n, m).
constexpr int BATCH_MAX = 16;
constexpr long long BATCH_MAP_WGS = 512;   // map workgroups of a launch of two or more matrices (see plan_batch_map)

struct BatchItem {
  const void* Y;
  void* X;
  void* ws;
  float* v_out;
  float* u_out;
  unsigned char* mask_out;
  long long n, m;
  double eta;
  int wide;   // the wide form of LaneCols (see wide_rows)
  int whole;  // one-kernel form: X overlaps Y, one workgroup does the whole matrix; chain: the map pass takes that form's search
};

struct BatchItems {
  int count;
  BatchItem item[BATCH_MAX];
};

struct BatchGrid {
  unsigned first[BATCH_MAX + 1];  // first workgroup of every problem in this launch, then the total
};

// Row groups of the map pass per column tile, for every problem of a launch.  Every map workgroup
// runs the whole threshold search of its problem, so their number is planned for the launch, not
// problem by problem: one by one, sixteen matrices of 1024 x 1024 made 4096 workgroups with a
// search and one block of 16 rows each.  Where the grids of the single calls come to at most 512 workgroups together they
// are kept.  Otherwise all problems get the same number of row blocks per
// workgroup, the smallest that keeps the launch within 512 workgroups (1024 where no matrix has more than 256 columns,
// whose search is one value per thread; twice the column tiles where those are more, so that a tall matrix beside wide
// ones is still shared).  Measured, us per batch with the single calls' grids / 256 / 512 / 1024 workgroups:
// 16 x (1024 x 1024) 55.3 / 46.3 / 45.2 / 44.4; 6 x (4096 x 4096) 209 / 224 / 201 / 205; 8 x (10000 x 256) 50.8 / 52.5 /
// 52.0 / 51.1; 300x5000 + 4000x64 + 77x900 + 2000x2000 36.8 / 26.3 / 25.5 / 27.8; 16384x4096 + 1024x1024 (512 in all) 126 /
// 143 / 135 / 136.
// (A row's result does not depend on the workgroup that maps it: the bits stay those of the
// single calls.)
struct BatchMapPlan {
  int groups[BATCH_MAX];
};
// tiles, rows, columns, own: of every problem; own: row groups of its single call.
static inline void plan_batch_map(int count, const long long* tiles, const long long* rows, const long long* columns,
                                  const long long* own, BatchMapPlan* plan) {
  long long all_tiles = 0, all_own = 0, most = 1, widest = 0;   // most: row blocks of the tallest matrix
  for (int i = 0; i < count; ++i) {
    all_tiles += tiles[i];
    all_own += tiles[i] * own[i];
    if (cdiv(rows[i], MAP_RBLK) > most) most = cdiv(rows[i], MAP_RBLK);
    if (columns[i] > widest) widest = columns[i];
  }
  if (all_own <= BATCH_MAP_WGS) {
    for (int i = 0; i < count; ++i) plan->groups[i] = (int)own[i];
    return;
  }
  long long target = widest <= WG ? 2 * BATCH_MAP_WGS : BATCH_MAP_WGS;
  if (target < 2 * all_tiles) target = 2 * all_tiles;
  long long lo = 1, hi = most;         // (the number of workgroups falls as blocks per workgroup rise; `most` always fits)
  while (lo < hi) {
    const long long blocks = lo + (hi - lo) / 2;
    long long wgs = 0;
    for (int i = 0; i < count; ++i) wgs += tiles[i] * cdiv(cdiv(rows[i], MAP_RBLK), blocks);
    if (wgs <= target) hi = blocks; else lo = blocks + 1;
  }
  for (int i = 0; i < count; ++i) plan->groups[i] = (int)cdiv(cdiv(rows[i], MAP_RBLK), lo);
}

// Row blocks that a map workgroup of a batch requests under its search (see colmap_body).  Every one costs 16 registers in
// fp32 and 32 on 16-bit storage, and the plan above counts on two workgroups per CU whatever the number of columns and on
// three up to 4096: as many as leave those.  One / four blocks, us: l1,inf fp32 16 x (1024 x 1024) 41.2 / 38.8, 4 x (512 x 6000) 35.7 / 33.5;
// bf16 28.0 / 29.5, 26.1 / 38.8 (one workgroup per CU).  l1,2 fp32 beyond 4096 columns has room for three: 4 x (512 x 6000)
// 35.0 / 33.9 with three / 37.8 with four, 16 x (1024 x 1024) 41.2 / 40.2 / 39.8; bf16 8 x (10000 x 256) 41.0 / 65.7.
template <int Q, typename T>
constexpr int map_ahead() {
  return sizeof(T) == 2 ? 1 : Q == QINF ? 4 : 3;
}

// The problem a workgroup belongs to, and its number within that problem.
__device__ __forceinline__ int batch_find(const BatchGrid& gr, int count, long long& bid) {
  int p = 0;
  while (p + 1 < count && blockIdx.x >= gr.first[p + 1]) ++p;
  bid = (long long)blockIdx.x - (long long)gr.first[p];
  return p;
}

template <int Q, typename T>
__global__ __launch_bounds__(WG) void colagg_batch_kernel(BatchItems it, BatchGrid gr) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  long long bid;
  const BatchItem& b = it.item[batch_find(gr, it.count, bid)];
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q));
  const T* Y = static_cast<const T*>(b.Y);
  if (b.wide) colagg_body<Q, T, WIDE, false>(Y, b.n, b.m, g, ws.partial, bid);
  else colagg_body<Q, T, WIDE, true>(Y, b.n, b.m, g, ws.partial, bid);
}

template <int Q, typename T>
__global__ __launch_bounds__(SWG) void reduce_batch_kernel(BatchItems it, BatchGrid gr) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  long long bid;
  const BatchItem& b = it.item[batch_find(gr, it.count, bid)];
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q));
  reduce_body<Q>(ws.partial, b.m, g, reduce_parts(g.groups, fold_threads(g.groups)), ws.v, b.v_out, ws.flags, bid);
}

// RIDE: some of the problems take the search of the one-kernel form (a build of its own: with both searches in every
// batch 16 x (1024 x 1024) takes 41.25 instead of 41.1 us).
template <int Q, typename T, int SC, bool RIDE = false>
__global__ __launch_bounds__(WG) void colmap_batch_kernel(BatchItems it, BatchGrid gr, BatchMapPlan mp, int outer) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  long long bid;
  const int p = batch_find(gr, it.count, bid);
  const BatchItem& b = it.item[p];
  Geometry g = plan_columns(b.n, b.m, WIDE, Q);
  g.map_groups = mp.groups[p];
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q));
  const T* Y = static_cast<const T*>(b.Y);
  T* X = static_cast<T*>(b.X);
  constexpr int SEARCH = Q == Q1 ? 0 : SC;   // l1,1: tau comes from the record, not from a search here
  constexpr int AHEAD = map_ahead<Q, T>();
  const double eta = b.eta;
  const int form = map_form(b.wide != 0, b.m, WIDE);
  const bool wave = RIDE && b.whole != 0;
  if (form == MAP_EVEN)
    colmap_body<Q, T, WIDE, MAP_EVEN, SEARCH, AHEAD>(Y, X, b.n, b.m, g, ws, b.u_out, b.mask_out, eta, outer, bid, wave);
  else if (form == MAP_RAGGED)
    colmap_body<Q, T, WIDE, MAP_RAGGED, SEARCH, AHEAD>(Y, X, b.n, b.m, g, ws, b.u_out, b.mask_out, eta, outer, bid, wave);
  else
    colmap_body<Q, T, WIDE, MAP_STRIDED, SEARCH, AHEAD>(Y, X, b.n, b.m, g, ws, b.u_out, b.mask_out, eta, outer, bid, wave);
}

// Matrices of at most 128 KiB each: the one-kernel form of tiny.h for all of them in one launch
// (up to 16 workgroups for a matrix whose X lies apart from Y, one for a matrix projected in place).
template <int Q, typename T>
__global__ __launch_bounds__(TINY_WG) void tiny_batch_kernel(BatchItems it, BatchGrid gr, int outer) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  long long bid;
  const BatchItem& b = it.item[batch_find(gr, it.count, bid)];
  TinyPlan tp;
  if (!tiny_plan(b.n, b.m, WIDE, &tp)) return;   // (the host only sends matrices that fit)
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q));
  tiny_body<Q, T, WIDE>(static_cast<const T*>(b.Y), static_cast<T*>(b.X), b.n, b.m, b.eta, outer, tp.cw, ws,
                           b.v_out, b.u_out, b.mask_out, bid, b.whole != 0);
}

// ------------------------------------------------------------------ l1,1: the inner searches
// The same for the kernels of the per-column threshold searches (l11.h).  Every problem has
// its own number of lock-step sweeps and hand-over count; a sweep kernel of the batch leaves
// the problems alone that planned fewer sweeps.
struct BatchL11Plan {
  int sweeps[BATCH_MAX];
  unsigned handoff[BATCH_MAX];
};

template <typename T, int SC>
__global__ __launch_bounds__(WG) void l11_init_batch_kernel(BatchItems it, BatchGrid gr, int outer) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  long long bid;
  const BatchItem& b = it.item[batch_find(gr, it.count, bid)];
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q1);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q1));
  l11_init_body<SC>(b.n, b.m, ws, b.eta, outer, bid);
}

template <typename T>
__global__ __launch_bounds__(WG) void l11_sweep_batch_kernel(BatchItems it, BatchGrid gr,
                                                             BatchL11Plan plan) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  __shared__ SweepLds<WAVE * WIDE> lds;
  long long bid;
  const int p = batch_find(gr, it.count, bid);
  if (plan.sweeps[p] < 1) return;
  const BatchItem& b = it.item[p];
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q1);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q1));
  const T* Y = static_cast<const T*>(b.Y);
  if (b.wide) l11_sweep_body<T, WIDE, false>(Y, b.n, b.m, g, ws, bid, lds);
  else l11_sweep_body<T, WIDE, true>(Y, b.n, b.m, g, ws, bid, lds);
}

template <typename T>
__global__ __launch_bounds__(WG) void l11_filter_batch_kernel(BatchItems it, BatchGrid gr,
                                                              BatchL11Plan plan, int sweep) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  __shared__ FilterLds<WAVE * WIDE> lds;
  long long bid;
  const int p = batch_find(gr, it.count, bid);
  if (sweep >= plan.sweeps[p]) return;
  const BatchItem& b = it.item[p];
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q1);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q1));
  const T* Y = static_cast<const T*>(b.Y);
  if (b.wide) l11_filter_body<T, WIDE, false>(Y, b.n, b.m, g, ws, sweep, plan.handoff[p], bid, lds);
  else l11_filter_body<T, WIDE, true>(Y, b.n, b.m, g, ws, sweep, plan.handoff[p], bid, lds);
}

template <typename T>
__global__ __launch_bounds__(WG) void l11_update_batch_kernel(BatchItems it, BatchGrid gr,
                                                              BatchL11Plan plan, int sweep) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  long long bid;
  const int p = batch_find(gr, it.count, bid);
  if (sweep >= plan.sweeps[p]) return;
  const BatchItem& b = it.item[p];
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q1);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q1));
  l11_update_body(b.n, b.m, g, ws, sweep, plan.handoff[p], bid);
}

template <typename T>
__global__ __launch_bounds__(FIN_WG) void l11_finish_batch_kernel(BatchItems it, BatchGrid gr,
                                                               BatchL11Plan plan) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  long long bid;
  const int p = batch_find(gr, it.count, bid);
  const BatchItem& b = it.item[p];
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q1);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q1));
  if (b.n <= (long long)FIN_ROWS * FIN_HELD)
    l11_finish_body<T, true>(static_cast<const T*>(b.Y), b.n, b.m, ws, plan.sweeps[p], plan.handoff[p], bid);
  else
    l11_finish_body<T, false>(static_cast<const T*>(b.Y), b.n, b.m, ws, plan.sweeps[p], plan.handoff[p], bid);
}

// l1,1 problems of at most 4096 rows after their aggregate pass: the columns-in-registers kernel
// of l11held.h, every workgroup running the outer search of its own problem.  NV: the values per
// thread the tallest problem of the launch needs.  EVEN as in l11_held_body, when it holds for every
// problem of the launch.  (Both bodies in one kernel: the two-per-CU builds spilled 42 to 48 registers
// instead of 19 to 29, every build held the LDS twice; 8 x (2048 x 2048) fp32 136 against 132 us.  A launch each
// for the even and the ragged problems of a mixed batch: 300x257 + 3 x (64x64) + 1000x512 40 against 25 us.)
// SC and COLS as in l11_held_body: the values of v per thread of the search (0: the record is read, see
// search_batch_kernel), and the columns of a stripe.
template <typename T, int NV, int SC, bool EVEN, bool PACKED = false, int COLS = LH_COLS>
__global__ __launch_bounds__(LH_WG, lh_min_waves(NV, PACKED)) void l11_held_batch_kernel(BatchItems it, BatchGrid gr,
                                                                                        int outer) {
  constexpr int WIDE = 16 / (int)sizeof(T);
  long long bid;
  const int p = batch_find(gr, it.count, bid);
  const BatchItem& b = it.item[p];
  const Geometry g = plan_columns(b.n, b.m, WIDE, Q1);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q1));
  const long long stripes = (long long)(gr.first[p + 1] - gr.first[p]);
  l11_held_body<T, NV, SC, COLS, EVEN, lh_windows(sizeof(T), PACKED)>(static_cast<const T*>(b.Y), static_cast<T*>(b.X), b.n, b.m, ws, b.u_out,
                                       b.mask_out, SC > 0 ? b.eta : -1.0, outer, stripe_of_workgroup(bid, stripes));
}

// The outer searches of l1,1 problems of 4097 to 16384 columns, one workgroup each: the search of a
// single call (search_kernel, same bits).
template <typename T>
__global__ __launch_bounds__(WG) void search_batch_kernel(BatchItems it, int outer) {
  __shared__ SearchScratch<WG / WAVE> s;
  const BatchItem& b = it.item[blockIdx.x];
  const Geometry g = plan_columns(b.n, b.m, 16 / (int)sizeof(T), Q1);
  const Ws ws = bind(b.ws, layout_for(g, b.m, Q1));
  const SearchOut o = search_block<WG, SEARCH_CACHE_BIG>(ws.v, b.m, b.eta, MODE_PROJECT, outer, s);
  if (threadIdx.x == 0) write_result(ws, o, nullptr);
}

}  // namespace mlproj

#endif
