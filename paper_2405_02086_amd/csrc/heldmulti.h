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
// norm has).  A workgroup that has polled `patience` times computes the missing slabs' norms itself,
// in the owner's order (so with the owner's bits), and posts them if they are still absent.  Every
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
// 53.0 us at 256 x 500 x 128 l1,1,1; with 64 chunks on 4 lanes the kernel spills.)
static inline void hm_layout(long long nvec, int* seg, int* kpf) {
  *seg = nvec <= 32 ? 4 : 16;
  const long long per_lane = cdiv(nvec, *seg);
  *kpf = per_lane <= 2 ? 2 : per_lane <= 4 ? 4 : per_lane <= 8 ? 8 : 16;
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
  // l1 fibres: the searches cost a workgroup the more the fuller its registers are, and the chain
  // spreads them over the whole chip: one pass only for lightly filled workgroups (64 x 200 x 64
  // l1,2: 15 against 18 us) or nearly a full grid (180 x 128 x 512: 33 against 43, 256^3 l1,1,1: 43.5
  // against 46.1; but 30 x 128 x 512 29 against 19, 150 x 60 x 1000 34 against 32, 64 x 400 x 64 24
  // against 21).
  const long long rounds = cdiv(spw * d1, nseg);
  if (q1 == Q1 && rounds * kpf > 8 && nwg < 176) return false;
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

}  // namespace mlproj

#endif
