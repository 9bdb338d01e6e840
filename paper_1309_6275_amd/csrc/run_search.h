// Index and threshold arithmetic of the road search on the layer runs
// (runs_kernel, reject_kernel), in integers only, so that the CPU tests compile
// and check the very lines that the kernels run.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define HT_RUN_FN __device__ __forceinline__
#else
#define HT_RUN_FN inline
#endif

namespace ht {

constexpr int kStage = 256;           // hits of a run staged at a time
constexpr int kVisit = 4;             // hits of a visit
// A hit's |f| and the number of its visit share a word, the number in the low
// bits: two arcs of kStage hits in whole visits.
constexpr uint32_t kVisitNum = 511u;
static_assert(2 * kStage <= (int)kVisitNum + 1, "every visited hit of a stage has a number");

// The end of the words of hits within thr: |f| <= thr has a word below it.  A word's
// low bits are not |f|'s, so the bound is thr rounded up (down, it lost the
// hits of the last 2^-14 before the road's edge); infinities and what is not a
// number stay at or beyond it.
HT_RUN_FN uint32_t road_words(uint32_t thr_bits) {
  const uint32_t end = (thr_bits | kVisitNum) + 1u;
  return end < 0x7f800000u ? end : 0x7f800000u;
}

// The three seed layers' listed members side by side over the lanes: the lane's
// seed layer s, the layer's first entry and entry count in the list, and the lane's
// entry.  A lane without one (s = -1, no entries) takes the first entry of layer 2,
// so that its entry's place is one of the run that it is looked up in.
struct SeedLane {
  int s, st, n, e;
};
HT_RUN_FN SeedLane seed_lane(int lane, int n0, int n1, int n2, int st0, int st1, int st2) {
  SeedLane v;
  int q = lane;
  v.s = -1;
  v.st = st2;
  v.n = 0;
  if (lane < n0) { v.s = 0; v.st = st0; v.n = n0; q = 0; }
  else if (lane < n0 + n1) { v.s = 1; v.st = st1; v.n = n1; q = n0; }
  else if (lane < n0 + n1 + n2) { v.s = 2; v.n = n2; q = n0 + n1; }
  v.e = v.st + lane - q;
  return v;
}
// the record of an entry of seed layer s (-1: of layer 2) whose place in the layer's
// run is the low half of hp; the runs begin at r0, r1 and r2
HT_RUN_FN int seed_record(int s, int r0, int r1, int r2, uint32_t hp) {
  return (s == 0 ? r0 : (s == 1 ? r1 : r2)) + (int)(hp & 0xffffu);
}

// The two arcs [a0, a1) and [b0, b1) of a lane's road, in order and at least a visit
// apart, so that no place is read for both (a hit visited twice would look like
// two, and one skipped for that reason would be lost): closer ones become one,
// with the hits between, whose visit changes nothing.
struct Arcs {
  int a0, a1, b0, b1;
};
HT_RUN_FN Arcs order_arcs(int a0, int a1, int b0, int b1) {
  const bool swap = b0 < b1 && b0 < a0;
  Arcs v;
  v.a0 = swap ? b0 : a0;
  v.a1 = swap ? b1 : a1;
  v.b0 = swap ? a0 : b0;
  v.b1 = swap ? a1 : b1;
  if (v.a0 < v.a1 && v.b0 < v.b1 && v.b0 < v.a1 + kVisit) {
    v.a1 = v.b1 > v.a1 ? v.b1 : v.a1;
    v.b0 = v.b1 = 0;
  }
  return v;
}
// A stage [g0, g0 + kStage) visits an arc from its first place there (a stage's
// visits start anew) while the place is below its end there.
HT_RUN_FN int stage_first(int begin, int g0) { return begin > g0 ? begin : g0; }
HT_RUN_FN int stage_end(int end, int g0) { return end < g0 + kStage ? end : g0 + kStage; }
// the place of the hit with number x, num1 numbers having gone to the first arc
HT_RUN_FN int visit_place(const Arcs& v, int g0, int x, int num1) {
  return x < num1 ? stage_first(v.a0, g0) + x : stage_first(v.b0, g0) + x - num1;
}

}  // namespace ht
