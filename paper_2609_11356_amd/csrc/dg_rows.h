// dg_rows.h -- device pieces shared by the row-reduction and normalisation
// kernels: one step of a leaf's fold, the wave-local LDS wait, and the
// count-down and count-up meetings of the lanes.
#pragma once

#include "dg_device.h"
#include "dg_internal.h"
#include "dg_lanes.h"

namespace dg {

__device__ __forceinline__ float leaf_step(float s, float x, int sumsq, int fma) {
  if (!sumsq) return s + x;
  if (fma) return __builtin_fmaf(x, x, s);
  float q = x * x;
  return s + q;
}

// The waves of a workgroup reduce different rows in disjoint LDS regions, so
// no workgroup barrier is needed: a wave waits for its own LDS operations
// (lgkmcnt(0)) before the next phase touches the same locations.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_wave_barrier();
}

// One step of a count-down butterfly over an array of per-lane values: each
// value meets its exact partner lane ^ M.
template <int M, int N>
__device__ __forceinline__ void down_step(float* s) {
#pragma unroll
  for (int u = 0; u < N; ++u) s[u] = s[u] + xor_partner<M>(s[u]);
}

// The count-down butterfly's lane steps over groups of G lanes: offsets
// G / 2, ..., 2, 1.
template <int G, int N>
__device__ __forceinline__ void down_lanes(float* s) {
  if constexpr (G >= 64) down_step<32, N>(s);
  if constexpr (G >= 32) down_step<16, N>(s);
  if constexpr (G >= 16) down_step<8, N>(s);
  if constexpr (G >= 8) down_step<4, N>(s);
  if constexpr (G >= 4) down_step<2, N>(s);
  if constexpr (G >= 2) down_step<1, N>(s);
}

// The lanes' partial results meet in the descriptor's tree (W lanes, leaf
// q LPL + u in lane q, slot u): leaf order = in-lane levels then the xor
// butterfly counting up; bit-reversed order = the butterfly counting down
// then the in-lane levels from the highest leaf bit.  Every lane ends with
// the result.
template <int LPL, bool DOWN>
__device__ __forceinline__ float lanes_meet(float (&s)[LPL]) {
  if constexpr (!DOWN) {
#pragma unroll
    for (int h = 1; h < LPL; h <<= 1)
#pragma unroll
      for (int u = 0; u < LPL; u += 2 * h) s[u] = s[u] + s[u + h];
    float r = s[0];
    return tree_sum_lanes<6>(r);
  } else {
    down_lanes<64, LPL>(s);
#pragma unroll
    for (int h = LPL / 2; h >= 1; h >>= 1)
#pragma unroll
      for (int u = 0; u < h; ++u) s[u] = s[u] + s[u + h];
    return s[0];
  }
}

}  // namespace dg
