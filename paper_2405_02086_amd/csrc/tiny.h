// mlproj: a whole bi-level projection in one kernel, for matrices of at most 128 KiB.
#ifndef MLPROJ_TINY_H
#define MLPROJ_TINY_H

#include "aggregate.h"
#include "common.h"
#include "reduce.h"
#include "search.h"

namespace mlproj {

// ------------------------------------------------------------------ tiny matrices
// A matrix this small costs three kernel launches and nothing else (13 us for 256 x 128).
// Here every workgroup reads ALL of Y into registers (16 chunks of 16 bytes per thread, 512
// threads: 128 KiB), folds the column aggregates through LDS in a fixed order, runs the
// threshold search (Eq. 6-7) itself, and then maps and stores its own share of the rows: the
// three steps of Alg. 1 with no hand-over between workgroups, so one launch.  All workgroups
// compute the same v and tau, bit for bit.  Reading Y sixteen times is served by the L2.
// The fp64 sums (of the search, for q = 2 also of the aggregate) are folded in another order than in
// the three-kernel chain, which can show in the last bit of an output; a batch sends the same
// matrices here as single calls do, so it still returns their bits.
//
// Threads form TINY_WG / cw row lanes of cw column lanes (cw = the chunks of a row, rounded up
// to a power of two); a thread holds rows tr, tr + rl, tr + 2 rl, ... of its chunk column, and
// workgroup b stores the rows of slot b.  That needs X apart from Y: a workgroup still reading Y
// would see rows another has already written.  When X overlaps Y (a projection in place, the
// usual call of a training loop) ONE workgroup does the whole matrix (`whole`): it has read all
// of Y into its registers before its first store, so any overlap is harmless, and the 128 KiB
// it then stores alone cost little beside the launches saved.
// Which forms are built: q = inf and q = 2.  (A q = 1 form, with the per-column searches of
// Alg. 3 run on the held registers, was built and dropped: on fp32 storage it took 43 us for a
// 256 x 128 matrix against 23 us for the general path, whose finishing pass spreads the columns
// over many workgroups instead of repeating every search in each; on 16-bit storage it needed 82 KB
// of LDS, all 256 registers and scratch memory, and its one run ended in a memory aperture fault.)
template <int Q, typename T>
constexpr bool tiny_built() { return Q != Q1; }

constexpr int TINY_WG = 512;
constexpr int TINY_WAVES = TINY_WG / WAVE;
constexpr int TINY_SLOTS = 16;            // rows per thread

struct TinyPlan {
  int cw;     // column lanes
  int rl;     // row lanes
  int slots;  // rows per thread in use = workgroups
};

// Whether an n x m matrix with `vec` elements per 16-byte chunk fits, and how.
__host__ __device__ static inline bool tiny_plan(long long n, long long m, int vec, TinyPlan* p) {
  if (m < vec || m > FUSED_SEARCH_MAX) return false;
  // (long ragged rows of 16-bit elements: the lanes' unaligned LDS accesses cost more than the second launch of the
  // chain, 8 x 4001 bf16 12.0 against 10.7 us; 16 x 2001 11.3 against 11.1, and 25 against 28 where the caller waits)
  if (vec == 8 && m % vec != 0 && m > 2048) return false;
  const long long cpr = cdiv(m, vec);
  if (cpr > TINY_WG) return false;
  int cw = 1;
  while (cw < cpr) cw *= 2;
  const int rl = TINY_WG / cw;
  const long long slots = cdiv(n, rl);
  if (slots > TINY_SLOTS) return false;
  p->cw = cw;
  p->rl = rl;
  p->slots = (int)slots;
  return true;
}

// (`bid` is the workgroup's number within its own problem: blockIdx.x for a single matrix.)
template <int Q, typename T, int VEC>
__device__ __forceinline__ void tiny_body(const T* Y, T* X, long long n,
                                          long long m, double eta, int outer, int cw, const Ws& ws,
                                          float* __restrict__ v_out, float* __restrict__ u_out,
                                          unsigned char* __restrict__ mask_out, long long bid,
                                          bool whole) {
  using Acc = typename AccOf<Q>::type;
  __shared__ alignas(16) Acc sm_part[TINY_WG * VEC];   // [row lane][column]
  __shared__ SearchScratch<TINY_WAVES> bs;
  // v (zero beyond column m) takes the place of row lane 0 of the partials, in their type (fp32
  // maxima are exact, sums stay fp64): column c of that row is read by the one thread that then
  // writes v_c, and the other rows lie behind it.  The partials are 8 to 32 KiB (q = 2 on 16-bit storage), the search's scratch 4.3.
  Acc* const sm_v = sm_part;
  static_assert(sizeof(Acc) * TINY_WG * VEC + sizeof(SearchScratch<TINY_WAVES>) <= 37 * 1024,
                "tiny_body: the partial aggregates of this (q, storage type) need more LDS than planned");
  const int rl = TINY_WG / cw;
  const int tc = threadIdx.x % cw;
  const int tr = threadIdx.x / cw;
  const long long cpr = cdiv(m, VEC);
  const bool col_ok = tc < cpr;
  // The chunk that would run past the end of the row is the row's last 16 bytes instead: its first
  // `shadow` elements are its neighbour's, aggregated there, and stored by both with the same
  // values (every element is in registers before the first store).  A lane without a chunk
  // shadows that last one.
  const long long at = ((long long)tc + 1) * VEC <= m ? (long long)tc * VEC : m - VEC;
  const int shadow = col_ok ? (int)(tc * VEC - at) : VEC;
  const int width = cw * VEC;
  const bool whole_chunks = VEC == 8 && m % VEC == 0;   // (the same for the whole workgroup; see below)

  Pack<T, VEC> raw[TINY_SLOTS];
#pragma unroll
  for (int k = 0; k < TINY_SLOTS; ++k) {
    const long long row = tr + (long long)k * rl;
    raw[k] = load_pack<T, VEC>(Y + (row < n ? row : n - 1) * m + at);
  }
  __builtin_amdgcn_sched_barrier(0);
  Acc acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = (Acc)0;
#pragma unroll
  for (int k = 0; k < TINY_SLOTS; ++k) {
    if (tr + (long long)k * rl < n) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) accumulate<Q>(acc[e], (float)raw[k].e[e]);
    }
  }
  // Fold over the row lanes: those of a wavefront on the crossbar (a column has WAVE / cw of them there),
  // what is left, at most a row per wavefront or row lane, through LDS.
  for (int o = cw; o < WAVE; o *= 2) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = combine<Q>(acc[e], __shfl_xor(acc[e], o));
  }
  const bool lanes_meet = cw < WAVE;
  const int rows = lanes_meet ? TINY_WAVES : rl;
  const int my_row = lanes_meet ? (int)threadIdx.x / WAVE : tr;
  // (Whole chunks of 16-bit elements in wide LDS accesses, here and below: element by element, eight lanes meet on
  // every bank; 8 x 4096 bf16 10.8 against 10.4 us.  fp32 gains nothing, and a batch of 15 fp32 l1,2 matrices took 25.4
  // instead of 24.6.)
  if (!lanes_meet || (int)(threadIdx.x & (WAVE - 1)) < cw) {
    if (whole_chunks) {   // (columns past the end included: nobody reads what is made of them)
#pragma unroll
      for (int e = 0; e < VEC; ++e) sm_part[my_row * width + tc * VEC + e] = acc[e];
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e)
        if (e >= shadow) sm_part[my_row * width + at + e] = acc[e];
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < width; c += TINY_WG) {
    Acc a = sm_part[c];
    for (int r = 1; r < rows; ++r) a = combine<Q>(a, sm_part[r * width + c]);
    const double vj = (Q == Q2) ? sqrt((double)a) : (double)a;
    sm_v[c] = c < m ? (Acc)vj : (Acc)0;
  }
  __syncthreads();

  // Few groups: every wavefront searches for itself (16 x (256 x 128) in a batch: 11.0 -> 9.2 us
  // with the fold above).
  const SearchOut o = m <= WAVE_SEARCH_MAX
      ? search_wave<WAVE_SEARCH_CACHE, Acc>(sm_v, (int)m, eta, outer)
      : search_block<WG, SEARCH_CACHE, TINY_WG, Acc>(sm_v, m, eta, MODE_PROJECT, outer, bs);
  const Top top = top_of(o);
  if (bid == 0) {
    if (threadIdx.x == 0) write_result(ws, o, nullptr);
    for (long long c = threadIdx.x; c < m; c += TINY_WG) {
      const double uj = radius((double)sm_v[c], top);
      if (v_out) v_out[c] = (float)sm_v[c];
      if (u_out) u_out[c] = (float)uj;
      if (mask_out) mask_out[c] = uj > 0.0 ? 1 : 0;
    }
  }
  float uf[VEC];
  double par[VEC];   // q = 2: scale u_j / v_j
  Acc mine[VEC];
  if (whole_chunks) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) mine[e] = sm_v[tc * VEC + e];
  } else {
#pragma unroll
    for (int e = 0; e < VEC; ++e) mine[e] = sm_v[at + e];
  }
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    const double vj = (double)mine[e];
    const double uj = radius(vj, top);
    uf[e] = (float)uj;
    par[e] = (Q == Q2 && vj > 0.0) ? uj / vj : 0.0;
  }
  if (!col_ok) return;
  // this workgroup's rows: slot `bid` of every thread (every slot when it works alone)
#pragma unroll
  for (int k = 0; k < TINY_SLOTS; ++k) {
    if (whole || k == (int)bid) {
      const long long row = tr + (long long)k * rl;
      if (row < n) {
        Pack<T, VEC> f;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float y = (float)raw[k].e[e];
          if constexpr (Q == QINF) f.e[e] = (T)copysignf(fminf(fabsf(y), uf[e]), y);
          else f.e[e] = round_to<T>((double)y * par[e]);
        }
        store_pack(X + row * m + at, f);
      }
    }
  }
}

template <int Q, typename T, int VEC>
__global__ __launch_bounds__(TINY_WG) void tiny_kernel(const T* Y, T* X,
                                                       long long n, long long m, double eta,
                                                       int outer, int cw, Ws ws,
                                                       float* __restrict__ v_out,
                                                       float* __restrict__ u_out,
                                                       unsigned char* __restrict__ mask_out,
                                                       int whole) {
  tiny_body<Q, T, VEC>(Y, X, n, m, eta, outer, cw, ws, v_out, u_out, mask_out, blockIdx.x, whole != 0);
}

}  // namespace mlproj

#endif
