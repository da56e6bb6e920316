// Device helpers of the kernels that work on one matrix row per group of
// lanes (a power of two up to a wavefront) with the row staged in LDS.
#pragma once

#include "common.hpp"

namespace airg {

// Orders this wavefront's LDS accesses before and after the call.  A group
// never spans wavefronts, and a wavefront's LDS operations execute in order,
// so no barrier is needed.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The group's lanes among a wavefront ballot, lane 0 of the group in bit 0.
template <int G>
__device__ __forceinline__ unsigned long long group_ballot(bool b) {
  const unsigned long long m = __ballot(b);
  if constexpr (G == 64) return m;
  const int first = (int)(threadIdx.x & 63) & ~(G - 1);
  return (m >> first) & ((1ull << (G & 63)) - 1ull);
}
__device__ __forceinline__ int bits_below(unsigned long long m, int lane) {
  return (int)__popcll(m & ((1ull << lane) - 1ull));
}

// Lanes per row for rows of avg entries on average, and the LDS capacity per
// row that goes with it (rows past it take a slow path in global memory):
// 24 KB of columns and values per workgroup of 256 for the short rows, 48 KB
// for the longest, so that three to six workgroups fit a CU.
#define AIRG_ROW_GROUPS(avg, CALL) \
  do {                             \
    if ((avg) <= 3.0) {            \
      CALL(4, 32);                 \
    } else if ((avg) <= 10.0) {    \
      CALL(8, 64);                 \
    } else if ((avg) <= 28.0) {    \
      CALL(16, 128);               \
    } else if ((avg) <= 96.0) {    \
      CALL(32, 512);               \
    } else {                       \
      CALL(64, 1024);              \
    }                              \
  } while (0)

}  // namespace airg
