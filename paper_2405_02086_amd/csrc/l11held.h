// mlproj: bi-level l1,1 (Alg. 3) for matrices of at most 4096 rows, columns kept in registers.
#ifndef MLPROJ_L11HELD_H
#define MLPROJ_L11HELD_H

#include "common.h"
#include "l11.h"
#include "reduce.h"
#include "search.h"

namespace mlproj {

// ------------------------------------------------------------------ l1,1 from registers
// Alg. 3 after the column sums: the outer threshold, then for every kept column the threshold
// tau_j with sum_i max(|Y_ij| - tau_j, 0) = u_j, then X = sign(Y) max(|Y| - tau_j, 0).  The
// lock-step sweeps of l11.h read the whole matrix once per step because a column is strided in
// memory.  A matrix of at most 4096 rows lets one workgroup hold 16 whole columns instead (one
// 64-byte run of every row, as the finishing pass does): 512 threads x up to 128 elements.  The
// workgroup reads its stripe once, finds the thresholds on registers (no memory traffic per
// step), and maps and stores from the same registers: after the aggregate pass Y is read once
// and X written once, whatever the number of steps.
// What bounds it: loads, searches and stores are one chain in every workgroup (4096 x 4096, one per CU, time stamps: 13 us of loads
// with the outer search and the first evaluation under them, 8 us of steps, 11 us of stores), and an evaluation
// of all held entries costs 3 to 4 us there.  So as few of them as possible: the first is at the guess, every further one lists the
// entries of a window that should hold the root, and among those it is found exactly (two evaluations as a rule instead of
// three to eight; 4096 x 4096 54.1 -> 49.7 us per call, 2001 x 3003 38.0 -> 33.3).
//
// A lane owns VEC = 16 bytes' worth of neighbouring columns (one vector access per row), CW
// lanes span the stripe, and the thread of row lane r holds rows r, r + RL, r + 2 RL, ...  The
// partial sums and counts of a column are folded over the row lanes of a 16-lane row on the
// DPP crossbar (rotations by CW, 2 CW, ... 8), then over the 4 rows of each of the 8
// wavefronts through LDS by the 32 lanes that step the column, always in the same order, and
// the listed entries add up exactly in any order: the result repeats bit for bit.
constexpr int LH_WG = 512;
constexpr int LH_COLS = 16;
constexpr int LH_COLS_NARROW = 8;   // fp32, 4097 to 8192 rows: stripes of 8 columns (32-byte runs), 128 values per thread
constexpr int LH_WAVES = LH_WG / WAVE;
constexpr int LH_FOLD_ROWS = LH_WAVES * (WAVE / 16);   // partial rows per column in LDS
// The host sends larger matrices through the sweeps: 64M elements of fp32, 32M of a 16-bit type
// (whose 16-column stripes are 32-byte runs: 1024 x 65536 bf16 takes 0.34 ms here against 0.21).
template <typename T>
constexpr long long lh_max_elems() { return sizeof(T) == 4 ? (64LL << 20) : (32LL << 20); }
constexpr int DPP_ROR2 = 0x122;
constexpr int LH_SEARCH_CACHE = 8;   // values of v per thread when the kernel runs the outer search itself: up to 4096 columns

template <typename T, int COLS = LH_COLS>
struct LhShape {
  static constexpr int VEC = 16 / (int)sizeof(T);
  static constexpr int CW = COLS / VEC;
  static constexpr int RL = LH_WG / CW;
  static_assert(CW == 2 || CW == 4, "the crossbar fold is written for 2 or 4 lanes per run");
  static_assert(COLS <= LH_COLS, "the LDS arrays hold LH_COLS columns");
};

// values per thread a matrix of n rows needs (32, 64 or 128), 0 when it has too many rows
template <typename T>
static inline int lh_values_for(long long n) {
  const long long rows = (n + LhShape<T>::RL - 1) / LhShape<T>::RL * LhShape<T>::VEC;
  return rows <= 32 ? 32 : rows <= 64 ? 64 : rows <= 128 ? 128 : 0;
}
// ... and whether the narrow stripes (fp32 only) reach a matrix too tall for the wide ones
static inline bool lh_narrow_fits(long long n) {
  return (n + LhShape<float, LH_COLS_NARROW>::RL - 1) / LhShape<float, LH_COLS_NARROW>::RL * 4 <= 128;
}

// Whether a matrix takes the EVEN build of the kernel: every stripe of X begins and ends on a 64-byte sector, or
// rows are whole 16-byte pieces and so few that what their streamed stores leave half written costs less than
// ordinary stores do (even / ragged build, us: 3000 x 12 fp32 29.6 / 32.7, 4000 x 20 31.0 / 32.7, 4000 x 104 bf16 36.6 / 38.5,
// 4000 x 500 fp32 41.3 / 41.7; but 4000 x 1004 46.9 / 45.2, 4000 x 4004 100 / 78).
__host__ __device__ static inline bool lh_even_rows(const void* X, long long m, int elem_bytes) {
  const unsigned long long ends = reinterpret_cast<uintptr_t>(X) | (unsigned long long)(m * elem_bytes);
  return ends % 64 == 0 || (ends % 16 == 0 && m <= 512);
}

// Whether a matrix that the registers hold is left to the sweeps: fp32 rows of no whole 64-byte sectors, one workgroup
// per CU, and the 32M elements from which on the sweeps start from the grid (held / sweeps, us: 4096 x 8193
// 169 / 159, 2100 x 27963 331 / 259, 4096 x 16004 299 / 253; but 2048 x 24577, two workgroups per CU, 207 / 226,
// 4096 x 6145 131 / 180, and with X over Y, whose lines the stripes' stores then find cached, 4001 x 15001 and
// a copy of Y 312 / 336).
template <typename T>
static inline bool lh_left_to_grid(long long n, long long m, bool apart) {
  return sizeof(T) == 4 && apart && lh_values_for<T>(n) == 128 && m * (long long)sizeof(T) % 64 != 0 && n * m >= L11_GRID_ELEMS;
}

// The values per thread a whole l1,1 call on an n x m matrix takes this kernel with, 0 for a matrix that goes through the
// sweeps (apart: X lies apart from Y).  (Against the sweeps: ahead up to 64M elements, 57 against 97 us at 4096 x 4096, 108 against 146
// at 4096 x 8192, 219 against 227 at 4096 x 16384, and far ahead where most columns are dropped, whose
// stripes are not even read; behind at 128M.  Rows that are not 16-byte aligned: 38 against 65 us at 2001 x
// 3003, 21 against 27 at 1001 x 333.)
template <typename T>
static inline int lh_values(long long n, long long m, bool apart) {
  if (m < 16 / (int)sizeof(T) || n * m > lh_max_elems<T>() || lh_left_to_grid<T>(n, m, apart)) return 0;
  return lh_values_for<T>(n);
}

constexpr int LH_LIST = 128;            // window entries kept per column
constexpr int LH_LIST_SPAN = 40;        // ... and the most a window is laid out for
constexpr int LH_WINDOWS = 6;           // windows a column tries before it goes on in plain steps
constexpr int LH_HALF = 32;             // lanes that step one column

struct LhLds {
  double s[LH_COLS][LH_FOLD_ROWS + 1];
  unsigned k[LH_COLS][LH_FOLD_ROWS + 1];
  float list[LH_COLS][LH_LIST];   // the entries of the columns' windows, in any order
  unsigned listed[LH_COLS];
  float hi[LH_COLS];      // the columns' windows as published: the smallest float above the upper end
  float lo[LH_COLS];      // ... and above the lower
  unsigned open[LH_COLS];
  float th[LH_COLS];      // the thresholds as fp32 pairs (see colmap_body)
  float tl[LH_COLS];
};

// Sum over the lanes of a 16-lane row that own the same columns (the same lane % CW).
template <int CW>
__device__ __forceinline__ double lh_row_sum(double x) {
  if constexpr (CW <= 2) x += dpp_all_f64<DPP_ROR2>(x);
  x += dpp_all_f64<DPP_ROR4>(x);
  x += dpp_all_f64<DPP_ROR8>(x);
  return x;
}
template <int CW>
__device__ __forceinline__ unsigned lh_row_sum_u(unsigned x) {
  if constexpr (CW <= 2) x += dpp_u32<DPP_ROR2>(x);
  x += dpp_u32<DPP_ROR4>(x);
  x += dpp_u32<DPP_ROR8>(x);
  return x;
}
// max(a, |x|) for a >= 0 (fmaxf spends two more instructions on what it makes of signalling NaNs).
__device__ __forceinline__ float max_abs(float a, float x) {
  asm("v_max_f32 %0, %0, |%1|" : "+v"(a) : "v"(x));
  return a;
}
template <int CTRL>
__device__ __forceinline__ float max_with_dpp(float x) {
  return max_abs(x, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xf, 0xf, true)));
}
template <int CW>
__device__ __forceinline__ float lh_row_max(float x) {
  if constexpr (CW <= 2) x = max_with_dpp<DPP_ROR2>(x);
  x = max_with_dpp<DPP_ROR4>(x);
  return max_with_dpp<DPP_ROR8>(x);
}

// Sums and maxima over 32 lanes, the same bits in every one of them: in each step two lanes, or two groups of
// lanes that agree, exchange what they hold.
constexpr int DPP_HALF_MIRROR = 0x141, DPP_MIRROR = 0x140;
struct Halves { unsigned even, odd; };   // what the even and the odd one of two neighbouring 16-lane rows hold
__device__ __forceinline__ Halves rows_of(unsigned x) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return Halves{r[0], r[1]};
}
__device__ __forceinline__ double half_sum(double x) {
  x += dpp_all_f64<DPP_SWAP1>(x);
  x += dpp_all_f64<DPP_SWAP2>(x);
  x += dpp_all_f64<DPP_HALF_MIRROR>(x);
  x += dpp_all_f64<DPP_MIRROR>(x);
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  const Halves lo = rows_of((unsigned)b), hi = rows_of((unsigned)(b >> 32));
  return __longlong_as_double((long long)(((unsigned long long)hi.even << 32) | lo.even)) +
         __longlong_as_double((long long)(((unsigned long long)hi.odd << 32) | lo.odd));
}
__device__ __forceinline__ unsigned half_sum_u(unsigned x) {
  x += dpp_u32<DPP_SWAP1>(x);
  x += dpp_u32<DPP_SWAP2>(x);
  x += dpp_u32<DPP_HALF_MIRROR>(x);
  x += dpp_u32<DPP_MIRROR>(x);
  const Halves r = rows_of(x);
  return r.even + r.odd;
}
__device__ __forceinline__ float half_max(float x) {
  x = max_with_dpp<DPP_SWAP1>(x);
  x = max_with_dpp<DPP_SWAP2>(x);
  x = max_with_dpp<DPP_HALF_MIRROR>(x);
  x = max_with_dpp<DPP_MIRROR>(x);
  const Halves r = rows_of(__float_as_uint(x));
  return max_abs(__uint_as_float(r.even), __uint_as_float(r.odd));
}

// Whether a build lists windows or takes plain steps only.  A window saves one to three evaluations; it costs a comparison and two
// lane masks per value in every evaluation, and the listing.  Not with two workgroups of 64 values per CU on 16-bit storage, bound by
// instructions, where registers spill (20 to 30 with windows, 12 to 28 without) and eight columns of listing share a row.
// Windows / plain steps / the form before both, us at a radius of 0.2 norms, bf16: 2000 x 10000 Gaussian 63.1 / 64.8 / 63.8, Laplace 76.7 / 70.8 / 70.9; 2001 x
// 15003 93.0 / 91.7 / 90.1 and 109 / 100 / 100; 2048 x 8192 72.5 / 69.4 / 76.6 and 79.1 / 74.0 / 80.4; 1500 x 5000 42.8 / 44.9 / 44.5 and 50.8 / 48.9 /
// 48.5; 8 x (2048 x 2048) in a batch 113 / 112 / 108 and 120 / 113 / 112.  (Sums of 16-bit entries within a factor 2^33 are exact
// in 64 bits: either way a column ends with the same threshold.)
constexpr bool lh_windows(int elem_bytes, bool packed) { return !(elem_bytes == 2 && packed); }

// NV: values per thread (rows per thread x VEC).  SC > 0: every workgroup runs the outer search
// itself (SC values of v per thread), workgroup 0 files the result record; SC = 0: a search
// kernel ran before and the record is read.  X may alias Y: a thread writes only elements it has read, and
// what it reads beside them (see below) goes nowhere.
// WINDOWS: see lh_windows.
// EVEN: every stripe's runs lie on whole 64-byte sectors of X (lh_even_rows); otherwise rows may start
// anywhere.  (Two builds: with the ragged form's tests and stores beside it the even one lost 1 to 2 %.)
template <typename T, int NV, int SC, int COLS, bool EVEN, bool WINDOWS>
__device__ __forceinline__ void l11_held_body(const T* Y, T* X, long long n, long long m, const Ws& ws,
                                              float* __restrict__ u_out, unsigned char* __restrict__ mask_out,
                                              double seed_eta, int outer, long long bid) {
  using Sh = LhShape<T, COLS>;
  constexpr int VEC = Sh::VEC, CW = Sh::CW, RL = Sh::RL;
  constexpr int ROWS = NV / VEC;
  __shared__ LhLds lds;
  __shared__ SearchScratch<LH_WAVES> bs;
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  const int wave = tid / WAVE;
  const int cw = tid % CW;            // which 16-byte piece of the stripe's run
  const int rl = tid / CW;            // row lane
  // The stripe is COLS whole columns.  Ragged rows: the last stripe ends with the row and overlaps the
  // stripe before it (in a row shorter than a stripe the last lanes overlap their neighbours instead;
  // m >= VEC).  The overlap is loaded and summed like the rest.  Lanes of one workgroup that overlap (m < COLS) hold
  // the same values and file the same sums; columns of the stripe before belong to another workgroup, which in place may be
  // storing them meanwhile: what comes of them reaches no threshold (no lanes here own them, so nothing opens or
  // steps them), no loop exit and no store.  Even rows: a lane past the end shadows the last columns and stores nothing.
  const long long own0 = bid * COLS;                 // first column the workgroup owns
  const long long s0 = EVEN || own0 + COLS <= m ? own0 : (m < COLS ? 0 : m - COLS);   // first column of the stripe
  const long long want = s0 + (long long)cw * VEC;
  const long long col0c = (EVEN ? want < m : want + VEC <= m) ? want : m - VEC;   // the lane's columns: col0c .. col0c + VEC - 1
  const int lc = EVEN ? cw * VEC : (int)(col0c - s0);         // ... and their place in the stripe
  const long long mine0 = want > own0 ? want : own0;
  const int skip = EVEN ? (want < m ? 0 : VEC) : mine0 - col0c < VEC ? (int)(mine0 - col0c) : VEC;   // leading columns somebody else owns
  // Byte offsets of the thread's elements from the start of the matrix, in 32 bits (the host
  // sends at most lh_max_elems<T>() elements here): one address register per access instead of two.
  const unsigned off0 = (unsigned)(((long long)rl * m + col0c) * (long long)sizeof(T));
  const unsigned step = (unsigned)((long long)RL * m * (long long)sizeof(T));
  const unsigned off_last = (unsigned)(((n - 1) * m + col0c) * (long long)sizeof(T));
  const char* const ybytes = reinterpret_cast<const char*>(Y);

  // the stripe, as stored, every load in flight at once (a row past the end re-reads the last one)
  Pack<T, VEC> raw[ROWS];
  auto request_rows = [&](auto first, auto last) {   // (compile-time bounds: raw[] must stay in registers)
#pragma unroll
    for (int u = decltype(first)::value; u < decltype(last)::value; ++u) {
      const unsigned off = rl + u * RL < (int)n ? off0 + (unsigned)u * step : off_last;
      raw[u] = load_pack<T, VEC>(reinterpret_cast<const T*>(ybytes + off));
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // The rows are asked for in parts: a wavefront stops at a load that the memory pipeline has no room for, and with it
  // everything its workgroup has to do meanwhile.  With the search inside (rows behind its loads of v / ahead of its rounds too, us): 4096 x
  // 4096 4 / 12 50.4, 8 / 8 51.0, 8 / 16 50.0, 8 / 24 50.0, all 32 at once 54.6; 2001 x 3003 4 / 12 33.4, 8 / 8 33.7, 8 / 16 34.5.  (Eleven shapes of 500 to 8192 rows, fp32 and bf16: 4 / 4 everywhere is
  // within 2 %, but 1500 x 3000 28.2 / 27.7, 8192 x 1024 60.1 / 57.0 and the other way 3500 x 3501 49.0 / 49.8, 6000 x 2000 77.2 / 78.5.)  With
  // the search ahead: the first quarter at once, the rest when the stripe is known to be needed.
  constexpr int EARLY = SC > 0 ? (ROWS <= 16 ? 4 : 8) : (ROWS >= 4 ? ROWS / 4 : 1);
  constexpr int MIDDLE = SC > 0 ? (ROWS <= 8 ? ROWS : ROWS <= 16 ? 12 : 16) : ROWS;
  using R0 = std::integral_constant<int, 0>;
  using RE = std::integral_constant<int, EARLY>;
  using RM = std::integral_constant<int, MIDDLE>;
  using RN = std::integral_constant<int, ROWS>;

  // Stores the lane's own columns of its rows: value(u, k) for row u, column k.  Even rows are streamed
  // past the caches.  Ragged runs end in two partly written sectors each, which the neighbouring
  // stripes (on the same XCD, see stripe_of_workgroup) complete: ordinary stores, so that the L2 can
  // merge them (2001 x 3003: 38 against 48 us).  (The offset and the row are made opaque in
  // each branch: formed ahead of both, the addresses and row tests of all rows would sit in registers
  // beside the held data, which then spill.)
  auto store_rows = [&](auto value) {
    const int rows = (int)n;
    if constexpr (EVEN) {
      if (skip != 0) return;
      unsigned at = off0;
      int row = rl;
      asm volatile("" : "+v"(at), "+v"(row));
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        if (row + u * RL < rows) {
          float f[VEC];
#pragma unroll
          for (int k = 0; k < VEC; ++k) f[k] = value(u, k);
          store_row<VEC, true>(reinterpret_cast<T*>(reinterpret_cast<char*>(X) + (at + (unsigned)u * step)), f);
        }
      }
    } else {
      unsigned at = off0;
      int row = rl;
      if (skip == 0) {
        asm volatile("" : "+v"(at), "+v"(row));
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
          if (row + u * RL < rows) {
            float f[VEC];
#pragma unroll
            for (int k = 0; k < VEC; ++k) f[k] = value(u, k);
            store_row<VEC, false>(reinterpret_cast<T*>(reinterpret_cast<char*>(X) + (at + (unsigned)u * step)), f);
          }
        }
      } else {
        asm volatile("" : "+v"(at), "+v"(row));
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
          if (row + u * RL < rows) {
            T* p = reinterpret_cast<T*>(reinterpret_cast<char*>(X) + (at + (unsigned)u * step));
#pragma unroll
            for (int k = 0; k < VEC; ++k)
              if (k >= skip) store_one_nt(p + k, (T)value(u, k));
          }
        }
      }
    }
  };

  // The 32 lanes that step column c of the stripe: half wavefront c of the workgroup.
  const int hc = tid / LH_HALF, hl = tid % LH_HALF;
  const long long j = s0 + hc;
  const bool owner = hc < COLS && (EVEN || j >= own0) && j < m;
  const long long jj = owner ? j : 0;
  double vj = 0.0;

  Top top;
  bool inside, nothing;
  if constexpr (SC > 0) {
    // (the search runs under a part of the stripe; the column sum is requested ahead of all, since loads return in order)
    if (owner) vj = ws.v[jj];
    __builtin_amdgcn_sched_barrier(0);
    const SearchOut o = search_block<LH_WG, SC, LH_WG, double>(ws.v, m, seed_eta, MODE_PROJECT, outer, bs,
                                                                      [&]() { request_rows(R0(), RE()); }, [&]() { request_rows(RE(), RM()); });
    top = top_of(o);
    inside = o.inside != 0u;
    nothing = inside || o.active == 0u;
    if (bid == 0 && tid == 0) {
      write_result(ws, o, nullptr);
      ws.res->inner_finished = nothing ? 0u : o.active;
    }
  } else {
    // (the record and the column sums are requested ahead of the rows: loads return in order)
    mlproj_result* res = ws.res;
    top = top_of(res);
    inside = res->inside_ball != 0u;
    const unsigned n_active = res->n_active;
    if (owner) vj = ws.v[jj];
    __builtin_amdgcn_sched_barrier(0);
    request_rows(R0(), RE());
    nothing = inside || n_active == 0u;
    if (bid == 0 && tid == 0) res->inner_finished = nothing ? 0u : n_active;
  }

  // The column's radius, bounds and state (the same in its 32 lanes).
  double uj = 0.0, lb = 0.0, t = 0.0;
  bool mine = false, open = false;
  if (owner) {
    uj = radius_of(ws, jj, vj, top);
    mine = !inside && uj > 0.0;
    open = mine;
    if (hl == 0) {
      if (u_out) u_out[j] = (float)uj;
      if (mask_out) mask_out[j] = uj > 0.0 ? 1 : 0;
    }
  }
  if constexpr (SC == 0) {
    // The search ran ahead, so the radii are known early: a stripe whose columns are all dropped
    // (the sparse results the projection is used for) is zeroed, and three quarters of it are
    // never read (the first quarter was requested with the radii, so that a stripe that is
    // needed does not wait twice).
    const bool need = inside || __syncthreads_or(uj > 0.0 ? 1 : 0) != 0;
    if (!need) {
      store_rows([](int, int) { return 0.0f; });
      return;
    }
    request_rows(RE(), RM());
  }
  // (the starting guess only now: with the search ahead, the rest of the stripe is on its way)
  // a dropped column maps to zero: threshold +inf; inside the ball nothing moves: threshold 0
  t = mine ? l11_guess(vj, uj, n, lb, HUGE_VALF) : (inside ? 0.0 : HUGE_VAL);   // (the same for a column somebody else owns)

  float held[ROWS][VEC];
  auto widen_row = [&](int u) {
    const bool row_ok = rl + u * RL < (int)n;
#pragma unroll
    for (int k = 0; k < VEC; ++k) held[u][k] = row_ok ? (float)raw[u].e[k] : 0.0f;   // |0| is never above a threshold
  };
  // What a lane found over its rows goes to LDS: first over the lanes of a 16-lane row.
  auto file_sums = [&](double (&s)[VEC], unsigned (&cnt)[VEC]) {
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
      s[k] = lh_row_sum<CW>(s[k]);
      cnt[k] = lh_row_sum_u<CW>(cnt[k]);
    }
    if ((lane & 15) < CW) {
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        lds.s[lc + k][wave * 4 + lane / 16] = s[k];
        lds.k[lc + k][wave * 4 + lane / 16] = cnt[k];
      }
    }
  };

  // First evaluation, at the guess, while the rows are still arriving: sum and count of the entries above it and the
  // columns' largest entries.  (Also where nothing is searched: a branch around it would have the rows in two places.)
  auto publish_threshold = [&]() {
    const float th = (float)t;
    lds.th[hc] = th;
    lds.tl[hc] = t < HUGE_VAL ? (float)(t - (double)th) : 0.0f;
  };
  if (hl == 0 && hc < COLS) {
    lds.hi[hc] = above(t);
    publish_threshold();   // (final where nothing is searched)
  }
  request_rows(RM(), RN());
  __syncthreads();
  float hm[VEC];
  double s[VEC];
  unsigned cnt[VEC];
  {
    float ct[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) { ct[k] = lds.hi[lc + k]; hm[k] = 0.0f; s[k] = 0.0; cnt[k] = 0u; }
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      widen_row(u);
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        const float h = fabsf(held[u][k]);
        const bool in = h >= ct[k];
        s[k] += (double)(in ? h : 0.0f);
        cnt[k] += in ? 1u : 0u;
        hm[k] = max_abs(hm[k], held[u][k]);
      }
#pragma unroll
      for (int k = 0; k < VEC; ++k) asm volatile("" : "+v"(s[k]), "+v"(cnt[k]), "+v"(hm[k]));   // (row by row: nothing is put off)
    }
  }

  if (!nothing) {
    file_sums(s, cnt);
#pragma unroll
    for (int k = 0; k < VEC; ++k) hm[k] = lh_row_max<CW>(hm[k]);
    if ((lane & 15) < CW) {
#pragma unroll
      for (int k = 0; k < VEC; ++k) lds.list[lc + k][wave * 4 + lane / 16] = hm[k];   // (no list yet)
    }
    __syncthreads();
    // The window of the next evaluation: (t, hi], or hi = t for a plain step.  With the sum and the count above a
    // point p, and e = S / K - p the mean excess there, entries lie about e / K apart and a Newton step of length d
    // from p ends about d^2 / (2 e) short of the root.  The window holds twice that and two entries; where that comes to
    // more than LH_LIST_SPAN entries the next step is a plain one (Laplace entries, 4000 x 3000, us: at most 12 entries
    // 58.3, 24 53.4, 40 53.5, without windows 56.4).
    double hi = HUGE_VAL;
    unsigned kprev = NO_COUNT;
    int windows = 0;
    bool certain = true;    // t is a lower bound on the root
    auto lay_window = [&](double S, unsigned K, double p) {
      hi = t;
      if constexpr (!WINDOWS) return;
      const float rk = __builtin_amdgcn_rcpf((float)K), d = (float)(t - p), e = (float)fma(-(double)K, p, S) * rk, gap = e * rk;
      const float width = d * d * __builtin_amdgcn_rcpf(e) + 2.0f * gap;
      if (K > 0u && e > 0.0f && width <= (float)LH_LIST_SPAN * gap && windows < LH_WINDOWS) {
        hi = fmin(t + (double)width, t + t);   // (within a factor 2 the sums of listed entries are exact, in any order)
        if (hi > t) ++windows;
        else hi = t;
      }
    };
    auto publish = [&]() {
      if (hl == 0 && hc < COLS) {
        lds.hi[hc] = open ? above(hi) : INFINITY;
        lds.lo[hc] = open ? above(t) : INFINITY;
        lds.listed[hc] = 0u;
        lds.open[hc] = open ? 1u : 0u;
        publish_threshold();
      }
    };
    if (hc < COLS) {   // (the same for a whole wavefront)
      const double S = half_sum(lds.s[hc][hl]);
      const unsigned K = half_sum_u(lds.k[hc][hl]);
      const float amax = half_max(lds.list[hc][hl]);
      if (mine) {
        // (a_max - u_j is a second certified lower bound: the largest entry alone sums to a_max - t; it lies next to the root
        // where the radius is small)
        const double g = t;
        lb = fmax(lb, (double)amax - uj);
        if (K > 0u) {
          t = fmax((S - uj) / (double)K, lb);
          lay_window(S, K, g);
        } else {
          // the guess lies beyond every entry: on to where entries spread evenly up to a_max would have the root
          t = fmax(lb, (double)amax - sqrt(2.0 * (double)amax * uj / (double)n));
          certain = t == lb;
          hi = t;
        }
      }
    }
    publish();
    __syncthreads();
    for (;;) {
      // Evaluation at the upper ends; the entries of the windows are listed.
      float ch[VEC], cl[VEC];
#pragma unroll
      for (int k = 0; k < VEC; ++k) {
        ch[k] = lds.hi[lc + k];
        cl[k] = k < skip ? INFINITY : lds.lo[lc + k];   // (a column's entries are listed by the lane that owns it)
        s[k] = 0.0;
        cnt[k] = 0u;
      }
#pragma unroll
      for (int u = 0; u < ROWS; ++u) {
        unsigned long long listed[VEC], any = 0ull;   // lane masks
#pragma unroll
        for (int k = 0; k < VEC; ++k) {
          asm volatile("" : "+v"(held[u][k]));   // keeps the widening to fp64 in the loop: hoisted, it doubles the registers
          const float h = fabsf(held[u][k]);
          const bool in = h >= ch[k];
          s[k] += (double)(in ? h : 0.0f);
          cnt[k] += in ? 1u : 0u;
          if constexpr (WINDOWS) {
            listed[k] = __ballot(h >= cl[k]) & ~__ballot(in);
            any |= listed[k];
          }
        }
#pragma unroll
        for (int k = 0; k < VEC; ++k) asm volatile("" : "+v"(s[k]), "+v"(cnt[k]));   // (the sums are not put off beyond the branch)
        if (WINDOWS && any != 0ull) {   // (one entry in some hundreds)
          unsigned found = 0u;
#pragma unroll
          for (int k = 0; k < VEC; ++k) found |= __builtin_amdgcn_inverse_ballot_w64(listed[k]) ? 1u << k : 0u;
          while (found != 0u) {
            const int k = __ffs(found) - 1;
            float h = held[u][0];
#pragma unroll
            for (int e = 1; e < VEC; ++e) h = k == e ? held[u][e] : h;
            const unsigned at = atomicAdd(&lds.listed[lc + k], 1u);
            if (at < (unsigned)LH_LIST) lds.list[lc + k][at] = fabsf(h);
            found &= found - 1u;
          }
        }
      }
      file_sums(s, cnt);
      __syncthreads();
      if (__any(open ? 1 : 0)) {   // (a wavefront whose columns are closed has no step to take)
        const double S = half_sum(lds.s[hc][hl]);
        const unsigned K = half_sum_u(lds.k[hc][hl]);
        const unsigned listed = lds.listed[hc];
        const bool window = WINDOWS && open && hi > t;
        const bool solve = window && listed <= (unsigned)LH_LIST;
        double tn = t;
        // Inside the window: the fixed point over the listed entries and what lies above them, from the bound t.
        float x[LH_LIST / LH_HALF];
#pragma unroll
        for (int q = 0; q < LH_LIST / LH_HALF; ++q) {
          const unsigned i = (unsigned)(hl + q * LH_HALF);
          x[q] = solve && i < listed ? lds.list[hc][i] : 0.0f;
        }
        bool going = solve;
        unsigned kk = NO_COUNT;
        while (WINDOWS && __any(going ? 1 : 0)) {
          const float c = above(t);
          double ls = 0.0;
          unsigned lk = 0u;
#pragma unroll
          for (int q = 0; q < LH_LIST / LH_HALF; ++q) {
            const bool in = x[q] >= c;
            ls += (double)(in ? x[q] : 0.0f);
            lk += in ? 1u : 0u;
          }
          ls = S + half_sum(ls);
          lk = K + half_sum_u(lk);
          if (going) {
            if (lk == 0u || lk == kk) {
              going = open = false;   // t came from this very active set: it is the root
            } else {
              kk = lk;
              tn = (ls - uj) / (double)lk;
              if (tn > hi) going = false;      // the root lies beyond the window
              else if (tn > t) t = tn;
              else going = open = false;       // no move left: t is the root, to rounding
            }
          }
        }
        if (open && window) {
          kprev = NO_COUNT;
          if (solve) {   // tn is a lower bound, and so is the step from the upper end
            const double p = hi;
            t = K > 0u ? fmax(tn, (S - uj) / (double)K) : tn;
            lay_window(S, K, p);
          } else {       // more entries than the list takes (ties): plain steps from here on
            if (K > 0u) t = fmax(t, (S - uj) / (double)K);
            windows = LH_WINDOWS;
            hi = t;
          }
        } else if (open && !certain) {
          // from any point the step ends at or left of the root
          const double p = t;
          certain = true;
          t = K > 0u ? fmax((S - uj) / (double)K, lb) : lb;
          lay_window(S, K, p);
        } else if (open) {
          if (K == 0u || K == kprev) {
            open = false;   // t came from this very active set: it is the root
          } else {
            const double p = t;
            kprev = K;
            tn = (S - uj) / (double)K;
            if (tn > t) t = tn;
            else open = false;   // no move left: t is the root, to rounding
            lay_window(S, K, p);
          }
        }
      }
      publish();
      __syncthreads();
      if (!__any(lds.open[tid % COLS] != 0u)) break;
    }
  }
  if (hl == 0 && mine) {
    ws.tauj[j] = t;
    ws.done[j] = 1u;
  }
  float th[VEC], tl[VEC];
#pragma unroll
  for (int k = 0; k < VEC; ++k) {
    th[k] = lds.th[lc + k];
    tl[k] = lds.tl[lc + k];
  }
  store_rows([&](int u, int k) { return copysignf(fmaxf((fabsf(held[u][k]) - th[k]) - tl[k], 0.0f), held[u][k]); });
}

// Registers: 32 values per thread leave room for two workgroups per CU, 128 for one.  64 fit two
// only with twelve to 28 registers spilled on 16-bit storage (fp32: none to four), which pays when there are more stripes than CUs (the
// second workgroup's loads and stores run under the first one's arithmetic: 42 against 52 us at
// 2048 x 8192) and costs when every stripe has a CU to itself (27 against 23 us at 2048 x 2048):
// PACKED picks the two-per-CU build.
constexpr int lh_min_waves(int nv, bool packed) { return nv <= 32 ? 4 : nv <= 64 ? (packed ? 4 : 2) : 2; }

template <typename T, int NV, int SC, bool EVEN, bool PACKED = false, int COLS = LH_COLS>
__global__ __launch_bounds__(LH_WG, lh_min_waves(NV, PACKED)) void l11_held_kernel(
    const T* Y, T* X, long long n, long long m, Ws ws, float* __restrict__ u_out,
    unsigned char* __restrict__ mask_out, double seed_eta, int outer) {
  l11_held_body<T, NV, SC, COLS, EVEN, lh_windows(sizeof(T), PACKED)>(Y, X, n, m, ws, u_out, mask_out, seed_eta, outer,
                                 stripe_of_workgroup(blockIdx.x, gridDim.x));
}

}  // namespace mlproj

#endif
