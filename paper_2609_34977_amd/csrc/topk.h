// The k largest of up to 64 * NV 32-bit keys held by one wave, without LDS or
// barriers: key i lives in lane i % 64, register i / 64.
//
// The k-th largest key is found bit by bit, from the top: every lane counts
// its keys at or above the candidate and one integer sum over the wave decides
// the bit.  (A ballot and a scalar population count per register and bit is
// fewer instructions but a chain of vector-to-scalar hand-overs: 16 us for 576
// keys.)  Keys equal to the k-th are taken in ascending index order.  A
// block-wide bitonic sort of the same keys costs a barrier per stage (55 stages
// for 576 keys, 19 us).
#pragma once

#include "common.h"

namespace spider {

template <int NV>
struct TopK {
  uint32_t t;  // every key above t is among the k largest
  int ties;    // how many keys equal to t are
};

// keys past the last index must be 0; keys of indices that do not take part
// may be 0 too if the caller excludes them from ties (a threshold of 0 with
// ties > 0 occurs only when every key that takes part is selected or equal 0).
template <int NV>
__device__ __forceinline__ TopK<NV> wave_kth_largest(const uint32_t (&key)[NV], int nv, int k) {
  uint32_t t = 0;
  for (int bit = 31; bit >= 0; --bit) {
    const uint32_t cand = t | (1u << bit);
    int c = 0;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      if (v % 16 == 0 && v >= nv) break;
      c += key[v] >= cand;
    }
    c = __builtin_amdgcn_readfirstlane(wave_sum_int(c));
    if (c >= k) t = cand;
    if (c == k) break;  // exactly k keys at or above t: lower bits change nothing
  }
  int above = 0;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    if (v % 16 == 0 && v >= nv) break;
    above += key[v] > t;
  }
  return {t, k - __builtin_amdgcn_readfirstlane(wave_sum_int(above))};
}

// Lanes below this one in a 64-lane mask.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __popcll(mask & ((1ull << (threadIdx.x & 63)) - 1ull));
}

}  // namespace spider
