// mlproj: the kernels of the one-pass multi-level projection (see heldmulti.h for the design).
#include "heldmulti.h"

#include "common.h"
#include "reduce.h"
#include "search.h"

namespace mlproj {

__global__ __launch_bounds__(WG) void hm_clear_kernel(unsigned long long* __restrict__ posts, int n) {
  const int i = blockIdx.x * WG + threadIdx.x;
  if (i < n) posts[i] = HM_ABSENT;
}

// The chunks of one fibre that a lane holds.  Every load is unconditional (a chunk that does not exist
// reads the fibre's first one, and is blanked); the elements a ragged last chunk shares with the one
// before it are blanked there too: 0 adds nothing to a norm and is never above a threshold.
template <typename T, int SEG, int KPF>
struct HmLane {
  static constexpr int VEC = 16 / (int)sizeof(T);
  int sl;
  __device__ __forceinline__ int at(const HmPlan& p, int k) const {   // element offset in the fibre
    const int i = sl + k * SEG;
    return i >= p.nvec ? 0 : (i == p.nvec - 1 ? p.len - VEC : i * VEC);
  }
  __device__ __forceinline__ int blank(const HmPlan& p, int k) const {   // leading elements that do not count
    const int i = sl + k * SEG;
    return i >= p.nvec ? VEC : (i == p.nvec - 1 ? p.dup : 0);
  }
  __device__ __forceinline__ void load(const HmPlan& p, const T* fibre, Pack<T, VEC> (&x)[KPF]) const {
#pragma unroll
    for (int k = 0; k < KPF; ++k) x[k] = load_pack<T, VEC>(fibre + at(p, k));
  }
  __device__ __forceinline__ void blank_out(const HmPlan& p, Pack<T, VEC> (&x)[KPF]) const {
    if (p.nvec == KPF * SEG && p.dup == 0) return;   // (the same for the whole grid)
#pragma unroll
    for (int k = 0; k < KPF; ++k) {
      const int b = blank(p, k);
#pragma unroll
      for (int e = 0; e < VEC; ++e) x[k].e[e] = e < b ? (T)0.0f : x[k].e[e];
    }
  }
};

// || fibre ||_q, the same in every lane of the segment for q = inf, lane 0's taken otherwise.
template <int Q, typename T, int SEG, int KPF>
__device__ __forceinline__ double hm_fibre_norm(const Pack<T, 16 / (int)sizeof(T)> (&x)[KPF]) {
  constexpr int VEC = 16 / (int)sizeof(T);
  if constexpr (Q == QINF) {
    float a = 0.0f;
#pragma unroll
    for (int k = 0; k < KPF; ++k)
#pragma unroll
      for (int e = 0; e < VEC; ++e) a = fmaxf(a, fabsf((float)x[k].e[e]));
    return seg_max<SEG>((double)a);
  } else {
    double a = 0.0;
#pragma unroll
    for (int k = 0; k < KPF; ++k)
#pragma unroll
      for (int e = 0; e < VEC; ++e) accumulate_d<Q>(a, (double)(float)x[k].e[e]);
    const double s = seg_sum<SEG>(a);
    return Q == Q2 ? sqrt(s) : s;
  }
}

// The q2-norm of d1 fibre norms in LDS, by one wavefront, always in this order.
__device__ __forceinline__ double hm_slab_norm(const double* v, int d1, int q2) {
  const int lane = threadIdx.x & (WAVE - 1);
  double a = 0.0;
  for (int i = lane; i < d1; i += WAVE) {
    const double x = v[i];
    a = q2 == QINF ? fmax(a, x) : q2 == Q1 ? a + x : fma(x, x, a);
  }
  if (q2 == QINF) return wave_max(a);
  a = wave_sum(a);
  return q2 == Q2 ? sqrt(a) : a;
}

// The radii of a slab's d1 fibres, by one wavefront: its fibre norms v (q2-norm nv) projected onto the
// q2-ball of radius r (the map and the steps of fibre_map_cached_kernel, from the threshold Gaussian entries would have).  Up to
// 2 * WAVE norms are read from LDS in every step; of more a lane keeps its first eight in registers (same order, same bits).  All in registers / all in
// LDS / by this rule, us: 2048 x 2 x 50 l1,1,1 14.5 / 13.9 / 14.2, 1000 x 20 x 77 17.4 / 17.1 / 17.2; 39 x 265 x 11 l1,inf,1 12.7 / 13.1 / 12.8, 200 x 600 x 16 14.3 /
// 15.8 / 14.4, 250 x 1000 x 24 l1,2,1 28.2 / 29.4 / 28.6.
__device__ __forceinline__ void hm_slab_radii(const double* v, double* out, int d1, int q2, double nv, double r) {
  const int lane = threadIdx.x & (WAVE - 1);
  double par = 0.0;
  if (q2 == Q2) {
    par = nv > r ? r / nv : 1.0;
  } else if (q2 == Q1 && nv > r) {
    if (!(r > 0.0)) {
      par = HUGE_VAL;
    } else {
      const double floor_t = (nv - r) / (double)d1;
      const float guess = (float)(nv / (double)d1) * 1.25331414f * gauss_z((float)(r * __builtin_amdgcn_rcp(nv)));
      bool first = (double)guess > floor_t;
      par = first ? (double)guess : floor_t;
      unsigned kprev = 0xffffffffu;
      auto search = [&](auto add_above) {
        for (;;) {
          double s = 0.0;
          unsigned c = 0;
          add_above(s, c);
          s = wave_sum(s);
          c = wave_sum_u(c);
          if (first) {
            kprev = c > 0u ? c : 0xffffffffu;
            par = c > 0u ? fmax((s - r) / (double)c, floor_t) : floor_t;
            first = false;
          } else if (c == 0u || c == kprev) {
            break;
          } else {
            kprev = c;
            const double t = (s - r) / (double)c;
            if (t > par) par = t;
          }
        }
      };
      auto from_lds = [&](int begin, double& s, unsigned& c) {
        for (int i = begin + lane; i < d1; i += WAVE) {
          const double x = v[i];
          if (x > par) { s += x; ++c; }
        }
      };
      if (d1 <= 2 * WAVE) {
        search([&](double& s, unsigned& c) { from_lds(0, s, c); });
      } else {
        constexpr int KEPT = 8;
        double kept[KEPT];
#pragma unroll
        for (int k = 0; k < KEPT; ++k) kept[k] = lane + k * WAVE < d1 ? v[lane + k * WAVE] : 0.0;   // (0 is never above a threshold)
        search([&](double& s, unsigned& c) {
#pragma unroll
          for (int k = 0; k < KEPT; ++k) {
            if (k * WAVE < d1 && kept[k] > par) { s += kept[k]; ++c; }
          }
          from_lds(KEPT * WAVE, s, c);
        });
      }
    }
  }
  for (int i = lane; i < d1; i += WAVE) {
    const double x = v[i];
    out[i] = q2 == QINF ? fmin(x, r) : q2 == Q2 ? x * par : fmax(x - par, 0.0);
  }
}

// (Keeps the widening of 16-bit elements where they are used: shared between the phases, or hoisted out
// of a search, it doubles the registers of the held data.)
template <typename T, int VEC, int KPF>
__device__ __forceinline__ void hm_keep_stored(Pack<T, VEC> (&x)[KPF]) {
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int k = 0; k < KPF; ++k) {
      unsigned w[4];
      __builtin_memcpy(w, &x[k], 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(w[i]));
      __builtin_memcpy(&x[k], w, 16);
    }
  }
}

// max(d, 0) with the sign of x, d rounded to fp32 and then to the storage type.
template <typename T>
__device__ __forceinline__ T round_to_signed(double d, float x) {
  float f = copysignf(fmaxf((float)d, 0.0f), x);
  if constexpr (sizeof(T) == 2) asm("" : "+v"(f));   // (see round_to)
  return (T)f;
}

// Sum of fp32 values over the lanes of a segment (4 or 16 lanes): for steps that need no more.
template <int SEG>
__device__ __forceinline__ float hm_seg_sum_f(float x) {
  auto step = [&](auto ctrl) { x += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true)); };
  step(std::integral_constant<int, DPP_SWAP1>());
  step(std::integral_constant<int, DPP_SWAP2>());
  if constexpr (SEG == 16) {
    step(std::integral_constant<int, 0x141>());   // mirror of 8 lanes
    step(std::integral_constant<int, 0x140>());   // mirror of 16 lanes
  }
  static_assert(SEG == 4 || SEG == 16, "segments of a quad or a row");
  return x;
}

// above() of l11.h, without its test for an infinite t in the serial part of every step: that t gives a NaN here, and
// nothing is above it either way (there an infinite bound has to compare as a number).
__device__ __forceinline__ float hm_above(double t) {
  const float f = (float)t;
  return (double)f <= t ? __uint_as_float(__float_as_uint(f) + 1u) : f;
}

template <int Q, typename T, int SEG, int KPF>
__global__ __launch_bounds__(HM_WG) void held_multi_kernel(const void* Yv, void* Xv, HmPlan p, int q2, double eta, int outer, Ws ws,
                                                           unsigned long long* posts, float* __restrict__ v_out,
                                                           float* __restrict__ u_out, unsigned patience) {
  constexpr int VEC = 16 / (int)sizeof(T);
  const T* const Y = static_cast<const T*>(Yv);
  T* const X = static_cast<T*>(Xv);
  constexpr int ROUNDS = hm_slots((int)sizeof(T)) / KPF;
  constexpr int NSEG = HM_WG / SEG;
  static_assert(NSEG * ROUNDS <= HM_MAX_FIBRES, "norms and radii of every held fibre fit their LDS arrays");
  __shared__ double sm_v[HM_MAX_FIBRES];   // fibre norms
  __shared__ double sm_r[HM_MAX_FIBRES];   // ... their radii (a helper's scratch before that)
  __shared__ double sm_w[HM_MAX_SLABS];    // slab norms, of the whole tensor
  __shared__ SearchScratch<HM_WAVES> bs;
  __shared__ unsigned char sm_missing[HM_MAX_WGS], sm_list[HM_MAX_WGS];
  static_assert(HM_MAX_WGS <= 256, "a workgroup's number fits a byte");
  __shared__ unsigned sm_any;
  __shared__ int sm_left, sm_start;
  const int tid = threadIdx.x;
  const int wave = tid / WAVE, lane = tid & (WAVE - 1);
  const int seg = tid / SEG;
  const HmLane<T, SEG, KPF> hl{tid % SEG};
  const int wg = blockIdx.x;
  const int slab0 = wg * p.spw;
  const int slabs = p.d0 - slab0 < p.spw ? p.d0 - slab0 : p.spw;
  const int fibres = slabs * p.d1;
  const long long origin = (long long)slab0 * p.d1 * p.len;

  // 1. the share, into registers (a fibre that does not exist reads the last one)
  Pack<T, VEC> d[ROUNDS][KPF];
#pragma unroll
  for (int j = 0; j < ROUNDS; ++j) {
    if (j < p.rounds) {
      const int f = j * NSEG + seg;
      hl.load(p, Y + origin + (long long)(f < fibres ? f : fibres - 1) * p.len, d[j]);
    }
  }
  __builtin_amdgcn_sched_barrier(0);

  // 2. the norms of its fibres and slabs; the slabs' are posted
#pragma unroll
  for (int j = 0; j < ROUNDS; ++j) {
    if (j < p.rounds) {
      hl.blank_out(p, d[j]);
      const double v = hm_fibre_norm<Q, T, SEG, KPF>(d[j]);
      const int f = j * NSEG + seg;
      if (hl.sl == 0 && f < fibres) sm_v[f] = v;
    }
  }
  __syncthreads();
  for (int s = wave; s < slabs; s += HM_WAVES) {
    const double w = hm_slab_norm(sm_v + s * p.d1, p.d1, q2);
    if (lane == 0)
      __hip_atomic_exchange(posts + slab0 + s, (unsigned long long)__double_as_longlong(w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // 3. everybody's slab norms
  constexpr int WORDS = HM_MAX_SLABS / HM_WG;
  unsigned taken = 0u;      // which of this thread's words are in sm_w
  bool complete = false;
  for (int round = 0; round < HELD_MAX_ROUNDS && !complete; ++round) {
    if (tid == 0) sm_any = 0u;
    if (tid < HM_MAX_WGS) sm_missing[tid] = 0;
    __syncthreads();
    for (unsigned spins = 0;; ++spins) {
      bool all = true;
#pragma unroll
      for (int i = 0; i < WORDS; ++i) {
        const int a = tid + i * HM_WG;
        if (a < p.d0 && !(taken & (1u << i))) {
          const unsigned long long x = __hip_atomic_load(posts + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (x != HM_ABSENT) {
            sm_w[a] = __longlong_as_double((long long)x);
            taken |= 1u << i;
          } else {
            all = false;
          }
        }
      }
      if (__all(all) || spins >= patience) break;
      __builtin_amdgcn_s_sleep(8);
    }
#pragma unroll
    for (int i = 0; i < WORDS; ++i) {
      const int a = tid + i * HM_WG;
      if (a < p.d0 && !(taken & (1u << i))) {
        sm_missing[a / p.spw] = 1;
        sm_any = 1u;
      }
    }
    __syncthreads();
    complete = sm_any == 0u;
    if (!complete) {
      // The shares still missing, listed.  Those that run (the others, as far as anyone can see) divide them: a
      // workgroup starts with its own section of the list, goes on around it, and looks at a share's words
      // once more before it computes it.
      if (wave == 0) {
        int n = 0, below = 0;   // missing so far; ... with a number below this workgroup's
        for (int g0 = 0; g0 < p.nwg; g0 += WAVE) {
          const bool miss = g0 + lane < p.nwg && sm_missing[g0 + lane] != 0;
          const unsigned long long all = __ballot(miss);
          if (miss) sm_list[n + __popcll(all & ((1ull << lane) - 1ull))] = (unsigned char)(g0 + lane);
          if (g0 <= wg && wg < g0 + WAVE) below = n + __popcll(all & ((1ull << (wg - g0)) - 1ull));
          n += __popcll(all);
        }
        if (lane == 0) {
          sm_left = n;
          sm_start = p.nwg > n ? (wg - below) * n / (p.nwg - n) : wg;
        }
      }
      __syncthreads();
      const int missing = sm_left, start = sm_start;
      for (int i = 0; i < missing; ++i) {
        const int g = sm_list[(start + i) % missing];   // (uniform)
        bool absent = false;
        for (int s = g * p.spw + tid; s < p.d0 && s < (g + 1) * p.spw; s += HM_WG)
          absent = absent || __hip_atomic_load(posts + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == HM_ABSENT;
        if (!__syncthreads_or(absent ? 1 : 0)) continue;
        // the share of workgroup g, its fibres and slabs normed in its own order
        const int g_slab0 = g * p.spw;
        const int g_slabs = p.d0 - g_slab0 < p.spw ? p.d0 - g_slab0 : p.spw;
        const int g_fibres = g_slabs * p.d1;
        const T* share = Y + (long long)g_slab0 * p.d1 * p.len;
        for (int j = 0; j < p.rounds; ++j) {
          const int f = j * NSEG + seg;
          Pack<T, VEC> x[KPF];
          hl.load(p, share + (long long)(f < g_fibres ? f : g_fibres - 1) * p.len, x);
          hl.blank_out(p, x);
          const double v = hm_fibre_norm<Q, T, SEG, KPF>(x);
          if (hl.sl == 0 && f < g_fibres) sm_r[f] = v;
        }
        __syncthreads();   // (every thread's reads of Y are behind it: see held.h for why the look comes after)
        for (int s = wave; s < g_slabs; s += HM_WAVES) {
          const double w = hm_slab_norm(sm_r + s * p.d1, p.d1, q2);
          unsigned long long* q = posts + g_slab0 + s;
          if (lane == 0 && __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == HM_ABSENT)
            __hip_atomic_exchange(q, (unsigned long long)__double_as_longlong(w), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
      }
    }
    __syncthreads();
  }

  // 4. tau, by every workgroup for itself
  // (few slabs: every wavefront for itself, without barriers)
  SearchOut o = p.d0 <= WAVE_SEARCH_MAX ? search_wave<WAVE_SEARCH_CACHE, double>(sm_w, p.d0, eta, outer)
                                        : search_block<WG, HM_MAX_SLABS / WG, HM_WG, double>(sm_w, p.d0, eta, MODE_PROJECT, outer, bs);
  if (!complete) o.tau = __longlong_as_double(0x7ff8000000000000LL);   // never reached: make it loud
  const Top top = top_of(o);
  if (wg == 0) {
    if (tid == 0) write_result(ws, o, nullptr);
    for (int a = tid; a < p.d0; a += HM_WG) {
      if (v_out) v_out[a] = (float)sm_w[a];
      if (u_out) u_out[a] = (float)radius(sm_w[a], top);
    }
  }

  // 5. the radii of the fibres
  for (int s = wave; s < slabs; s += HM_WAVES) {
    const double w = sm_w[slab0 + s];
    hm_slab_radii(sm_v + s * p.d1, sm_r + s * p.d1, p.d1, q2, w, radius(w, top));
  }
  __syncthreads();

  // 6. the fibres, from the registers.  (All loads are over.  Said here once: loads and stores share a counter, and the wait that
  // the compiler, for want of knowing, puts in front of a round's registers in the searches waits for the stores of the round
  // before.  256 x 256 x 256 l1,1,1: 41.7 -> 40.7 us; with 4 lanes per fibre it gains nothing and costs up to 2 %.)
  if constexpr (Q == Q1 && SEG == 16) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
  // (a little less than 1 / len: the all-active bound (nv - r) / len must not be rounded to the right of the root)
  const double per_element = (1.0 - 0x1p-51) / (double)p.len;
  // With 16 lanes per fibre the rounds go through the code in two passes, the second half of the registers moved to the first in
  // between: unrolled as a whole the two loops of the search, once per round, come to 90 KB, more than the instruction
  // cache, and a call that follows other kernels fetches them anew (256 x 256 x 256 l1,1,1 behind a product, a copy and an l1,1
  // projection 70 us, in two passes 61, repeated 39.3 / 38.9; what both replaced 64, repeated 43.8).
  constexpr int PASS = Q == Q1 && SEG == 16 && ROUNDS >= 4 ? ROUNDS / 2 : ROUNDS;
#pragma unroll 1
  for (int j0 = 0;;) {
#pragma unroll
    for (int j = 0; j < PASS; ++j) {
      if (j0 + j < p.rounds) {
        const int f = (j0 + j) * NSEG + seg;
        const int fc = f < fibres ? f : fibres - 1;
        const double nv = sm_v[fc], r = sm_r[fc];
        double par = 0.0;
        hm_keep_stored(d[j]);
        if constexpr (Q == Q2) par = nv > r ? r / nv : 1.0;
        if constexpr (Q == Q1) {
          // The fixed point of fibre_map_cached_kernel, on the elements as fp32: |x| > t is |x| >= above(t).  What the search costs is
          // vector instructions (the memory is idle meanwhile), so the steps far from the root are taken on fp32 sums, without a
          // quotient in fp64, until a step passes so few entries that the next one hardly passes any; and the last one is known
          // by no entry lying around it instead of by evaluating there once more.
          bool open = nv > r && r > 0.0 && f < fibres;
          const double floor_t = open ? (nv - r) * per_element : 0.0;
          if (nv > r && !(r > 0.0)) par = HUGE_VAL;
          // (floor_f rounded down: rounded up it may reach the entries of a fibre in which all are equal, and a search that starts there sees
          // none above it and ends: 256 x 256 x 256 ones at a radius of 0.1 came out as zeros)
          const float ratio = (float)(r * __builtin_amdgcn_rcp(nv)), rs = (float)r, floor_f = float_at_or_below(floor_t);
          float at = open ? fmaxf((float)(nv * per_element) * 1.25331414f * gauss_z(ratio), floor_f) : HUGE_VALF;
          if constexpr (SEG == 4 || KPF == 16) {
            // (16 fibres share a wavefront: what a step costs beside its elements counts little, and the fewest steps win.  16 chunks per lane
            // leave no registers, and their code no cache, for both loops: 200 x 30 x 1001 l1,1,1 24.9 / 23.9 us with this one alone,
            // 256 x 64 x 1024 35.9 / 36.7, behind other kernels 65.7 / 63.3)
            bool first = (double)at > floor_t;
            par = open ? (first ? (double)at : floor_t) : par;
            unsigned kfull = 0u;
            while (__any(open)) {
              const float ct = hm_above(par);
              double s = 0.0;
              unsigned c = 0;
              hm_keep_stored(d[j]);
#pragma unroll
              for (int k = 0; k < KPF; ++k)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                  const float h = fabsf((float)d[j][k].e[e]);
                  const bool in = h >= ct;
                  s += (double)(in ? h : 0.0f);
                  c += in ? 1u : 0u;
                }
              s = seg_sum<SEG>(s);
              c = seg_sum_u<SEG>(c);
              const double t = (s - r) / (double)c;
              if (open) {
                if (first) {
                  kfull = c;
                  par = c > 0u ? fmax(t, floor_t) : floor_t;
                } else if (c == 0u || c == kfull) {
                  open = false;
                } else {
                  kfull = c;
                  if (t > par) par = t;
                }
              }
              first = false;
            }
          } else {
            float bound = floor_f, margin = 0.0f;
            bool rough = open;
            unsigned kprev = 0u;
            for (int step = 0; step < 6 && __any(rough); ++step) {
              float s = 0.0f;
              unsigned c = 0;
              hm_keep_stored(d[j]);
#pragma unroll
              for (int k = 0; k < KPF; ++k)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                  const float h = fabsf((float)d[j][k].e[e]);
                  const bool in = h > at;
                  s += in ? h : 0.0f;
                  c += in ? 1u : 0u;
                }
              s = hm_seg_sum_f<SEG>(s);
              c = seg_sum_u<SEG>(c);
              if (rough) {
                const float rc = __builtin_amdgcn_rcpf((float)c), moved = (float)c - (float)kprev;
                // (from any point the step ends at or left of the root, and 64 fp32 additions are off by less than the margin, subnormal
                // sums included; a point beyond every entry says nothing: back towards the bound)
                if (c > 0u) {
                  margin = fmaf(8e-6f * s, rc, 1e-43f);
                  at = bound = fmaxf((s - rs) * rc - margin, floor_f);
                  rough = moved * moved > (float)c;
                } else {
                  at = fmaxf(0.6f * at, floor_f);
                }
                kprev = c;
              }
            }
            if (open) par = fmax((double)bound, floor_t);
            // (t is the root if it came from the active set of a point left of it and no entry lies between: the fp32 steps have
            // left a window (par, end] that holds it more often than not, and the entries of the window show in the same pass)
            double end = par + (double)(2.0f * margin);
            bool first = true;
            unsigned kfull = 0u;
            while (__any(open)) {
              const float ct = hm_above(par), ce = hm_above(end);
              double s = 0.0;
              unsigned c = 0;
              unsigned long long between = 0ull;   // lanes with an entry in the window
              hm_keep_stored(d[j]);
#pragma unroll
              for (int k = 0; k < KPF; ++k)
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                  const float h = fabsf((float)d[j][k].e[e]);
                  const bool in = h >= ct;
                  s += (double)(in ? h : 0.0f);
                  c += in ? 1u : 0u;
                  between |= __ballot(in) ^ __ballot(h >= ce);
                  asm volatile("" : "+s"(between));   // (at once: put off, the masks of all elements spill)
                }
              s = seg_sum<SEG>(s);
              c = seg_sum_u<SEG>(c);
              const bool clear = ((between >> (lane & ~(SEG - 1))) & ((1ull << SEG) - 1ull)) == 0ull;
              if (open) {
                if (c == 0u || c == kfull) {
                  open = false;
                } else {
                  const double t = (s - r) / (double)c;
                  const bool inside = clear && t >= par && t <= end;
                  open = !inside && (first || t > par);
                  if (first || t > par) par = fmax(t, floor_t);   // (the first may step back)
                  end = par + (double)(2.0f * margin);
                  kfull = c;
                }
              }
              first = false;
            }
          }
          hm_keep_stored(d[j]);
        }
        const float rf = (float)r;
        T* out = X + origin + (long long)fc * p.len;
#pragma unroll
        for (int k = 0; k < KPF; ++k) {
          Pack<T, VEC> z;
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            const float x = (float)d[j][k].e[e];
            if constexpr (Q == QINF) z.e[e] = (T)copysignf(fminf(fabsf(x), rf), x);
            else if constexpr (Q == Q2) z.e[e] = round_to<T>((double)x * par);
            else z.e[e] = round_to_signed<T>((double)fabsf(x) - par, x);
          }
          const int b = f < fibres ? hl.blank(p, k) : VEC;
          if (b == 0) {
            store_pack(out + hl.at(p, k), z);
          } else if (b < VEC) {
#pragma unroll
            for (int e = 0; e < VEC; ++e)
              if (e >= b) store_one_nt(out + hl.at(p, k) + e, z.e[e]);
          }
        }
      }
    }
    j0 += PASS;
    if (PASS == ROUNDS || j0 >= p.rounds) break;
#pragma unroll
    for (int j = 0; j < PASS && PASS + j < ROUNDS; ++j) {
#pragma unroll
      for (int k = 0; k < KPF; ++k) d[j][k] = d[PASS + j][k];
    }
  }
}

template <int Q, typename T, int SEG>
static HmKernel with_kpf(int kpf) {
  if (kpf == 4) return held_multi_kernel<Q, T, SEG, 4>;
  if (kpf == 8) return held_multi_kernel<Q, T, SEG, 8>;
  if constexpr (SEG == 4) {
    if (kpf == 2) return held_multi_kernel<Q, T, SEG, 2>;
  } else if constexpr (sizeof(T) == 4) {
    if (kpf == 16) return held_multi_kernel<Q, T, SEG, 16>;
  }
  return nullptr;
}
template <int Q, typename T>
static HmKernel with_seg(int seg, int kpf) {
  return seg == 4 ? with_kpf<Q, T, 4>(kpf) : seg == 16 ? with_kpf<Q, T, 16>(kpf) : nullptr;
}
template <int Q>
static HmKernel with_storage(int storage, int seg, int kpf) {
  switch (storage) {
    case MLPROJ_STORE_F32: return with_seg<Q, float>(seg, kpf);
    case MLPROJ_STORE_BF16: return with_seg<Q, bf16_t>(seg, kpf);
    default: return with_seg<Q, f16_t>(seg, kpf);
  }
}

HmKernel hm_kernel(int q1, int storage, int seg, int kpf) {
  return q1 == QINF ? with_storage<QINF>(storage, seg, kpf) : q1 == Q1 ? with_storage<Q1>(storage, seg, kpf) : with_storage<Q2>(storage, seg, kpf);
}
HmClear hm_clear() { return hm_clear_kernel; }

}  // namespace mlproj
