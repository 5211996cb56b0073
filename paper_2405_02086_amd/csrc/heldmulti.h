// mlproj: the multi-level projection with two inner levels in one pass over memory, for tensors the
// register files hold.
#ifndef MLPROJ_HELDMULTI_H
#define MLPROJ_HELDMULTI_H

#include "common.h"
#include "held.h"

namespace mlproj {

// ------------------------------------------------------------------ held fibres
// MP^nu (Sec. 5.2, Alg. 6) on a tensor (d0, d1, len) with inner norms q1 (of the fibres of len
// elements) and q2 (of the d1 fibre norms of a slab), one kernel instead of the chain of fibre.h (two
// aggregates, two maps): as in held.h a workgroup loads its share of Y ONCE and keeps it in registers
// (512 threads x 32 chunks of 16 bytes), but its share is whole slabs, so everything below the top
// level stays in the workgroup: the fibre norms and their radii in LDS, the fibres in registers.
// Only the slabs' norms travel.  What bounds it: 8 bytes of traffic per fp32 element instead of 12,
// and between the last load and the first store one exchange, the outer search and the map of the
// slab's norms; the in-register l1 searches of the fibres run under the stores of the fibres before
// them.  Measured, chain / one pass: see run_multilevel.
//
// Meeting.  As in held.h, with one 64-bit word per slab: its norm, an absent one all ones (a NaN no
// norm has).  A workgroup that has polled `patience` times computes missing slabs' norms itself,
// in the owner's order (so with the owner's bits), and posts those still absent.  The workgroups that run
// divide the missing shares among themselves.  (Every one of them going through all of them, 256 KiB of reading
// each, made 256^3 l1,1,1 on four streams take 327 to 347 us per projection where the streams ran at once;
// divided, 41 to 90.  The chain takes 33 to 37 there, but 48 against 46 alone.  l1,2,2: 311 to 325 / 28 to 60, chain 31
// to 34.  Beside a stream of matrix products as well: 372 to 602 / 344 to 351, chain 304.)  Every
// wait is bounded and everything waited for can be produced alone; in place is as safe as there, for
// the same reasons.
constexpr int HM_WG = HELD_WG;
constexpr int HM_WAVES = HM_WG / WAVE;
// Chunks a thread holds: 32 of fp32.  16-bit elements are widened for every phase, and with 16 chunks or
// more the kernel spills and loses to the chain (256^3 bf16 l1,1,1: 55 against 46 us): 8.
constexpr int hm_slots(int elem_bytes) { return elem_bytes == 4 ? HELD_SLOTS : 8; }
constexpr int HM_MAX_FIBRES = 2048;      // per workgroup (LDS: norms and radii, 32 KiB)
constexpr int HM_MAX_SLABS = 2048;       // of the tensor (LDS: 16 KiB)
constexpr int HM_MAX_WGS = 256;
constexpr unsigned long long HM_ABSENT = ~0ull;

struct HmPlan {
  int d0, d1, len;       // slabs, fibres per slab, elements per fibre
  int spw, nwg;          // slabs per workgroup, workgroups
  int nvec;              // 16-byte chunks of a fibre; when len is no multiple of them the last one is
  int dup;               // the fibre's last 16 bytes, and its first `dup` elements belong to the one before
  int rounds;            // fibres per segment
};

// SEG lanes hold a fibre with KPF chunks each.  (The elements cost the same either way, but every fold
// and every step of a fibre's search is paid per segment: 4 lanes beat 16 up to 32 chunks, 44.0 against
// 53.0 us at 256 x 500 x 128 l1,1,1; with 64 chunks on 4 lanes the kernel spills, 256^3 l1,1,1 44.8 against 40.6 us.)
static inline void hm_layout(long long nvec, int* seg, int* kpf) {
  *seg = nvec <= 32 ? 4 : 16;
  const long long per_lane = cdiv(nvec, *seg);
  *kpf = per_lane <= 2 ? 2 : per_lane <= 4 ? 4 : per_lane <= 8 ? 8 : 16;
}

// Whether one pass over memory beats the chain.  It has the traffic on its side (8 bytes per fp32 element
// against 12) and two launches against four, and three things against it: only its own workgroups work (the
// chain spreads a few large slabs over the whole chip), every chunk slot costs its arithmetic whether it holds
// elements or not, and a segment's streamed stores leave partly written 64-byte sectors where a fibre is no
// whole number of them.  The lines below were drawn on 4900 tensors of random sizes, radii and distributions on an
// MI355X (256 CUs): a class of tensors takes the one pass where its median is ahead of the chain's and its worst
// close to it.  What they sent here took 0.84 of the chain's time (geometric mean; 2.3 % of it was behind
// by more than 2 %), what they kept away would have taken 1.11.  The l1 searches of the fibres have become cheaper since, so a few of the l1 classes
// kept away would be level or ahead by now.  Chain / one pass, us, some of either kind (norms after the outer one innermost first):
//   taken    256^3 l1,2,2 39.1 / 29.5, l1,1,1 46.4 / 39.0; 6 x 71 x 64 l1,1,inf 14.1 / 10.3; 1000 x 128 x 81
//            l1,1,2 112 / 56; 256 x 64 x 1024 l1,2,2 39.3 / 33.7 (spilled registers and all, see below), l1,1,1 47.0 / 36.7; 200 x 30 x 1001 l1,1,1 37.4 / 24.0
//   refused  1 x 64 x 1000 l1,2,2 14.2 / 19.0 (one workgroup); 64 x 64 x 1000 l1,2,2 15.3 / 21.2; 1000 x 128 x 72
//            l1,2,inf 31.9 / 37.1 (sectors, idle slots); 2000 x 256 x 15 l1,1,1 48.5 / 51.7; 4 x 512 x 8 bf16 l1,1,1 18.7 / 27.1;
//            but 1000 x 128 x 81 l1,2,1 59.7 / 56.6, 64 x 64 x 500 l1,1,1 17.9 / 17.6
// q1: norm of the fibres; fibres, rounds: of a workgroup; cus: compute units.
static inline bool hm_pays(int q1, int elem_bytes, long long len, long long nvec, int seg, int kpf, long long fibres,
                           long long rounds, long long nwg, int cus) {
  const bool f32 = elem_bytes == 4, l1 = q1 == Q1;
  const bool few = nwg * 4 < cus, half = nwg * 2 >= cus, most = nwg * 16 >= (long long)cus * 11;   // of the chip at work
  const long long slots = rounds * kpf;                       // chunk slots per thread that are worked through
  const bool ragged = len % (16 / elem_bytes) != 0;           // (the chain goes element by element there)
  const bool sectors = len * elem_bytes % 64 == 0;
  const bool filled = nvec * 2 > seg * kpf;                   // a fibre uses more than half of its segment's slots
  const double used = (double)(fibres * nvec) / (double)(rounds * (HM_WG / seg) * seg * kpf);
  if (kpf == (f32 ? 16 : 8)) {
    // the most chunks per lane: fp32 spills 29 to 36 registers here, 16-bit has one round only
    if (l1 && ragged) return most && used >= 0.25;
    if (f32) return most && slots == HELD_SLOTS && (l1 ? len % 8 == 0 : nvec == seg * kpf && sectors && used > 0.6);
    if (ragged) return most && seg == 16 && used >= 0.25;
    return sectors && !few && used >= (l1 ? 0.75 : 0.4);
  }
  if (!l1) {
    if (!f32) return slots <= 4 || !ragged || (kpf == 4 && !few) || (most && !filled);
    if (slots <= 8) return !(ragged && slots == 8 && kpf == 4 && seg == 4);
    if (few || (slots > 16 && seg == 16 && !half)) return false;
    return seg == 16 || kpf == 2 || sectors || (kpf == 4 && len % 8 == 0);
  }
  if (kpf == 2 && rounds > 1 && !filled) return most && (f32 ? !ragged && slots <= 8 : ragged && len > 16);
  if (!f32) return slots <= 4 ? !(ragged && (rounds > 1 || (kpf == 4 && seg == 4))) || !few : most && (ragged || kpf == 4);
  if (slots <= 4) return true;
  if (slots <= 8) return kpf == 2 ? most : !few || !ragged || (seg == 16 && kpf == 8);
  if (!most) return false;
  if (kpf == 2) return ragged || nvec >= 7;
  return seg == 16 || kpf == 8 || sectors || (ragged && (slots <= 12 || len <= 48));
}

static inline bool hm_plan(long long d0, long long d1, long long len, int elem_bytes, int cus, int q1, HmPlan* p) {
  const int vec = 16 / elem_bytes;
  if (len < vec || d0 > HM_MAX_SLABS || d1 > HM_MAX_FIBRES) return false;
  const long long nvec = cdiv(len, vec);
  if (nvec > 256) return false;
  int seg, kpf;
  hm_layout(nvec, &seg, &kpf);
  if (cus > HM_MAX_WGS) cus = HM_MAX_WGS;
  if (cus <= 0) return false;
  const long long spw = cdiv(d0, (long long)cus);
  const long long nseg = HM_WG / seg;
  if (spw * d1 > nseg * (hm_slots(elem_bytes) / kpf)) return false;
  const long long nwg = cdiv(d0, spw);
  const long long rounds = cdiv(spw * d1, nseg);
  if (!hm_pays(q1, elem_bytes, len, nvec, seg, kpf, spw * d1, rounds, nwg, cus)) return false;
  p->d0 = (int)d0; p->d1 = (int)d1; p->len = (int)len;
  p->spw = (int)spw; p->nwg = (int)nwg;
  p->nvec = (int)nvec; p->dup = (int)(nvec * vec - len);
  p->rounds = (int)rounds;
  return true;
}

// One kernel for every q1, element type and layout, compiled in a translation unit of its own
// (heldmulti.hip); a null pointer for a layout that is not built.
typedef void (*HmKernel)(const void* Y, void* X, HmPlan p, int q2, double eta, int outer, Ws ws, unsigned long long* posts,
                         float* v_out, float* u_out, unsigned patience);
typedef void (*HmClear)(unsigned long long* posts, int n);
HmKernel hm_kernel(int q1, int storage, int seg, int kpf);
HmClear hm_clear();

// The kernel and plan of a tensor that takes the one pass (q1: norm of its fibres), null for one that does not.
static_assert((int)MLPROJ_NORM_INF == QINF && (int)MLPROJ_NORM_L1 == Q1 && (int)MLPROJ_NORM_L2 == Q2, "norms and kernel variants share their numbers");
static inline HmKernel hm_route(int storage, int q1, long long d0, long long d1, long long len, int cus, HmPlan* p) {
  if (!hm_plan(d0, d1, len, storage == MLPROJ_STORE_F32 ? 4 : 2, cus, q1, p)) return nullptr;
  int seg, kpf;
  hm_layout(p->nvec, &seg, &kpf);
  return hm_kernel(q1, storage, seg, kpf);
}

}  // namespace mlproj

#endif
