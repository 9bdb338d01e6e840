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

}  // namespace ht
