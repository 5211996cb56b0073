// mlproj: the map pass over columns (x_j = P^q_{u_j}(y_j), Eq. 8-9).
#ifndef MLPROJ_MAP_H
#define MLPROJ_MAP_H

#include "common.h"
#include "reduce.h"
#include "search.h"

namespace mlproj {

// ------------------------------------------------------------------ per-column map
// x_j = P^q_{u_j}(y_j) (Eq. 8-9) with u_j = max(v_j - tau, 0) (tau w_j for a weighted l1 ball):
//   q = inf : X = sign(Y) min(|Y|, u_j)          (the symmetric clip; Sec. 4.1)
//   q = 2   : X = Y * u_j / v_j
//   q = 1   : X = sign(Y) max(|Y| - tau_j, 0)    with tau_j from the inner searches
// Row blocks are visited from the bottom up, the reverse of the aggregate pass, so the rows
// read last there (the ones most likely still cached) are read first here.  For q = 1 the pass before
// is a listing sweep, which itself runs bottom up after the aggregate pass, so the order is top down
// (both together: 9001 x 3003 l1,1 148.6 -> 146.3 us; 16384 x 16384 746 -> 742, hardly more than two runs differ).
// SC > 0: every workgroup first runs the threshold search itself (see search_block; SC values of v per thread) and
// workgroup 0 files the result record; SC = 0: a search kernel ran before and tau is read from it (a build of its own, which
// the search's registers do not hold back where a CU runs several workgroups).
// FORM: how a lane reaches its columns (see LaneCols).  MAP_EVEN: 16-byte accesses, m a multiple of
// VEC; MAP_RAGGED: 16-byte accesses, any m >= VEC; MAP_STRIDED: one element per access.  (The test
// for the ragged lane at every store costs 1 % where there is none: 35.6 against 35.9 us at 4096 x 4096.)
// `bid` is the workgroup's number within its own problem (blockIdx.x for a single matrix).
// wave_search: the search of the one-kernel form, for a matrix whose single call takes that (at most WAVE_SEARCH_MAX columns).
constexpr int MAP_EVEN = 0, MAP_RAGGED = 1, MAP_STRIDED = 2;

// The form of a matrix whose aggregate pass is `wide` (see wide_rows).  Ragged rows are not worth 16-byte stores where
// a large part of the workgroups have next to nothing to store: two column tiles of which the second is an eighth full
// or less, or one tile of 16-bit elements up to three eighths full (map pass, one element / 16 bytes, us: 30000 x 257
// fp32 20.8 / 24.3, x 285 21.1 / 25.2, x 297 21.2 / 21.0; 40000 x 575 bf16 36.0 / 46.8, x 590 35.6 / 32.1, x 127 17.3 /
// 20.8, x 180 18.0 / 19.1, x 201 19.3 / 19.1; three tiles: 30000 x 513 fp32 27.9 / 26.8).
__host__ __device__ static inline int map_form(bool wide, long long m, int vec) {
  if (!wide) return MAP_STRIDED;
  if (m % vec == 0) return MAP_EVEN;
  const long long tile = (long long)WAVE * vec;
  if (m < tile ? m * 8 <= tile * 3 : m < 2 * tile && (m - tile) * 8 <= tile) return MAP_STRIDED;
  return MAP_RAGGED;
}

template <int Q, typename T, int VEC, int FORM, int SC, int AHEAD>
__device__ __forceinline__ void colmap_body(const T* Y, T* X, long long n, long long m,
                                            const Geometry& g, const Ws& ws,
                                            float* __restrict__ u_out,
                                            unsigned char* __restrict__ mask_out,
                                            double fused_eta, int outer, long long bid,
                                            bool wave_search = false) {
  constexpr int TILE_W = WAVE * VEC;
  constexpr int U = MAP_UNROLL;
  __shared__ SearchScratch<WAVES> bs;
  const int lane = threadIdx.x & (WAVE - 1);
  const int wave = threadIdx.x / WAVE;
  const long long t = bid % g.tiles;
  const long long grp = bid / g.tiles;
  const LaneCols<T, VEC, FORM == MAP_STRIDED, FORM == MAP_EVEN> lc(t * TILE_W, lane, m);
  const bool col_ok = lc.any();

  // Row blocks of MAP_RBLK rows, bottom block first (q = 1: top block first); the last block may be ragged.
  const long long nblk = (n + MAP_RBLK - 1) / MAP_RBLK;
  constexpr bool DOWN = Q != Q1;
  long long b = DOWN ? nblk - 1 - grp : grp;
  const long long step = DOWN ? -g.map_groups : g.map_groups;
  auto inside_rows = [&](long long blk) { return DOWN ? blk >= 0 : blk < nblk; };
  // The two buffers hold the elements as stored: widening them here would put a use of the
  // loaded values, and with it the wait for them, ahead of the stores of the current block.
  Pack<T, VEC> x[U], y[U];
  auto load_block = [&](long long blk, Pack<T, VEC> (&dst)[U]) {
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const long long row = blk * MAP_RBLK + wave + (long long)r * WAVES;
      if (row < n) lc.load(Y + row * m, dst[r]);
    }
  };
  // The first block is requested before tau is known, so its latency hides the search.  AHEAD > 1: that many blocks, the first
  // behind the search's own loads and the others when those have arrived (asked for ahead of them they hold up the
  // wavefronts, and with them the search).  Batches: see map_ahead.  Single calls, one workgroup per CU and a band of
  // rows that should stay narrow, take one block: 4096 x 4096 35.0 with 1, 35.2 with 2, 35.6 us with 4.
  Pack<T, VEC> ahead[AHEAD > 1 ? AHEAD - 1 : 1][U];
  auto request_first = [&]() {
    if (col_ok && inside_rows(b)) load_block(b, x);
  };
  auto request_ahead = [&]() {
#pragma unroll
    for (int a = 0; a < AHEAD - 1; ++a) {
      const long long blk = b + (a + 1) * step;
      if (col_ok && inside_rows(blk)) load_block(blk, ahead[a]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  Top top;
  bool inside;
  if constexpr (SC > 0) {
    SearchOut o;
    if constexpr (AHEAD > 1) {
      o = wave_search ? search_wave<WAVE_SEARCH_CACHE, double>(ws.v, (int)m, fused_eta, outer, request_first, request_ahead)
                      : search_block<WG, SC, WG, double>(ws.v, m, fused_eta, MODE_PROJECT, outer, bs, request_first, request_ahead);
    } else {
      request_first();
      o = wave_search ? search_wave<WAVE_SEARCH_CACHE, double>(ws.v, (int)m, fused_eta, outer)
                      : search_block<WG, SC>(ws.v, m, fused_eta, MODE_PROJECT, outer, bs);
    }
    top = top_of(o);
    inside = o.inside != 0u;
    if (bid == 0 && threadIdx.x == 0) write_result(ws, o, nullptr);
  } else {
    request_first();
    top = top_of(ws.res);
    inside = ws.res->inside_ball != 0u;
  }
  if constexpr (Q == Q1) {
    // A tile whose columns are all dropped (with sparse results most tiles are) is zeroed
    // without reading the rest of it.
    if (!inside) {
      bool kept = false;
#pragma unroll
      for (int k = 0; k < VEC; ++k)
        if (lc.ok[k]) kept = kept || radius_of(ws, lc.col(k), ws.v[lc.col(k)], top) > 0.0;
      if (!__syncthreads_or(kept ? 1 : 0)) {
        if (grp == 0 && wave == 0) {
#pragma unroll
          for (int k = 0; k < VEC; ++k) {
            if (lc.ok[k] && u_out) u_out[lc.col(k)] = 0.0f;
            if (lc.ok[k] && mask_out) mask_out[lc.col(k)] = 0;
          }
        }
        if (col_ok) {
          Pack<T, VEC> zero;
#pragma unroll
          for (int k = 0; k < VEC; ++k) zero.e[k] = (T)0.0f;
          for (; inside_rows(b); b += step) {
#pragma unroll
            for (int r = 0; r < U; ++r) {
              const long long row = b * MAP_RBLK + wave + (long long)r * WAVES;
              if (row < n) lc.store_nt(X + row * m, zero);
            }
          }
        }
        return;
      }
    }
  }
  if (!col_ok) return;

  float uf[VEC];
  double par[VEC];  // q = 2: scale u_j / v_j;  q = 1: inner threshold tau_j
#pragma unroll
  for (int k = 0; k < VEC; ++k) {
    const double vj = lc.ok[k] ? ws.v[lc.col(k)] : 0.0;
    const double uj = lc.ok[k] ? radius_of(ws, lc.col(k), vj, top) : 0.0;
    uf[k] = (float)uj;
    if constexpr (Q == Q2) par[k] = vj > 0.0 ? uj / vj : 0.0;
    else if constexpr (Q == Q1) par[k] = inside ? 0.0 : ((uj > 0.0 && lc.ok[k]) ? ws.tauj[lc.col(k)] : HUGE_VAL);
    else par[k] = 0.0;
  }
  // q = 1: tau_j as an unevaluated fp32 pair, tau_j = th + tl to 2^-48 relative.  |y| - th is
  // exact while |y| <= 2 th (the only place cancellation can occur) and carries one fp32
  // rounding beyond that, so (|y| - th) - tl stays within two fp32 units of the fp64 result.
  float th[VEC], tl[VEC];
#pragma unroll
  for (int k = 0; k < VEC; ++k) {
    th[k] = (float)par[k];
    tl[k] = (Q == Q1 && par[k] < HUGE_VAL) ? (float)(par[k] - (double)th[k]) : 0.0f;
  }
  if (grp == 0 && wave == 0) {
    if (u_out) {
#pragma unroll
      for (int k = 0; k < VEC; ++k)
        if (lc.ok[k]) u_out[lc.col(k)] = uf[k];
    }
    if (mask_out) {  // the kept columns, decided where the radius is: in fp64
#pragma unroll
      for (int k = 0; k < VEC; ++k)
        if (lc.ok[k]) mask_out[lc.col(k)] = radius_of(ws, lc.col(k), ws.v[lc.col(k)], top) > 0.0 ? 1 : 0;
    }
  }

  auto apply = [&](float yv, int k) -> T {
    if constexpr (Q == QINF) return (T)copysignf(fminf(fabsf(yv), uf[k]), yv);
    else if constexpr (Q == Q2) return round_to<T>((double)yv * par[k]);
    else return (T)copysignf(fmaxf((fabsf(yv) - th[k]) - tl[k], 0.0f), yv);
  };

  auto store_block = [&](long long blk, const Pack<T, VEC> (&src)[U]) {
#pragma unroll
    for (int r = 0; r < U; ++r) {
      const long long row = blk * MAP_RBLK + wave + (long long)r * WAVES;
      if (row < n) {
        Pack<T, VEC> f;
#pragma unroll
        for (int k = 0; k < VEC; ++k) f.e[k] = apply((float)src[r].e[k], k);
        lc.store_nt(X + row * m, f);
      }
    }
  };
  // The blocks requested under the search; the loads of the pipeline's next one go out ahead of their stores.
  if constexpr (SC > 0 && AHEAD > 1) {
    const long long nb = b + AHEAD * step;
    if (inside_rows(nb)) load_block(nb, y);
    if (inside_rows(b)) store_block(b, x);
#pragma unroll
    for (int a = 0; a < AHEAD - 1; ++a) {
      const long long blk = b + (a + 1) * step;
      if (inside_rows(blk)) store_block(blk, ahead[a]);
    }
#pragma unroll
    for (int r = 0; r < U; ++r) x[r] = y[r];
    b = nb;
  }
  // Software pipeline: the next block's loads are issued first, then this block is mapped
  // and stored, and only then does the wavefront wait.  On gfx9 loads and stores share one
  // counter, so any wait for a load also waits for every store issued before it: the wait
  // must come after both have been issued, or the two never overlap.
  // X may alias Y: a thread writes only elements that it has read, and what it reads beside them (a ragged lane the
  // columns of its neighbour, perhaps of another workgroup, stored by now or not) goes nowhere.
  for (; inside_rows(b); b += step) {
    const long long nb = b + step;
    if (inside_rows(nb)) load_block(nb, y);
    store_block(b, x);
#pragma unroll
    for (int r = 0; r < U; ++r) x[r] = y[r];
  }
}

template <int Q, typename T, int VEC, int FORM, int SC, int AHEAD>
__global__ __launch_bounds__(WG) void colmap_kernel(const T* Y, T* X, long long n,
                                                    long long m, Geometry g, Ws ws,
                                                    float* __restrict__ u_out,
                                                    unsigned char* __restrict__ mask_out,
                                                    double fused_eta, int outer) {
  colmap_body<Q, T, VEC, FORM, SC, AHEAD>(Y, X, n, m, g, ws, u_out, mask_out, fused_eta, outer, blockIdx.x);
}

}  // namespace mlproj

#endif
