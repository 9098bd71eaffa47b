// dg_attn_tile.h -- device pieces shared by the attention kernels: operand
// types, the MFMA wrappers, lane-group exchanges, and the key order and LDS
// swizzles of transposed score tiles.
#pragma once

#include <type_traits>

#include "dg_device.h"
#include "dg_internal.h"

namespace dg {
namespace {

typedef short shortx8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4* lds_s4;

__device__ __forceinline__ floatx4 mfma(const shortx8& a, const shortx8& b, const floatx4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                 0, 0);
}

// Compile-time loop: f(std::integral_constant<int, I>) for I in [B, E).
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

typedef float floatx16 __attribute__((ext_vector_type(16)));

typedef __attribute__((address_space(3))) void* lds_void;

// A workgroup barrier without the fence that would drain the loads in flight.
__device__ __forceinline__ void barrier_nofence() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// s_waitcnt immediate for at most n outstanding vector-memory operations.
constexpr int vmcnt_only(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

__device__ __forceinline__ void mfma_to(floatx16& c, const shortx8& a, const shortx8& b) {
  c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ void mfma_to(floatx4& c, const shortx8& a, const shortx8& b) { c = mfma(a, b, c); }

// (a, b) -> ([a.lo, b.lo], [a.hi, b.hi]) over the wave's 32-lane halves.
__device__ __forceinline__ void halves_swap(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
  a = __builtin_bit_cast(float, (int)r[0]);
  b = __builtin_bit_cast(float, (int)r[1]);
}
// The same over the 16-lane rows of each half.
__device__ __forceinline__ void rows_swap(float& a, float& b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), false, false);
  a = __builtin_bit_cast(float, (int)r[0]);
  b = __builtin_bit_cast(float, (int)r[1]);
}

// Key of MFMA row r of a K tile, and the swizzle of the K and V rows in LDS
// (chunk c of row t at c ^ swz(t)): the 16 rows one K fragment read takes, and
// the rows a transposing V read takes, on distinct slots of a 256-byte window.
template <int RW>
__device__ __forceinline__ int key_of_row(int r) {
  if constexpr (RW == 32) return 16 * (r >> 4) + 8 * ((r >> 2) & 1) + 4 * ((r >> 3) & 1) + (r & 3);
  else return 8 * (r >> 2) + (r & 3);            // + 4 in the step's second tile
}
template <int RW, int DC>
__device__ __forceinline__ int k_swz(int t) {
  if constexpr (RW == 32) return DC == 16 ? (t & 15) : ((t >> 1) & 7);
  else return DC == 16 ? ((t & 3) | ((t >> 1) & 12)) : (((t >> 1) & 1) | ((t >> 2) & 6));
}
template <int RW, int DC>
__device__ __forceinline__ int v_swz(int t) {
  if constexpr (RW == 32) return DC == 16 ? ((t & 3) << 2) : (((t >> 1) & 1) << 2);
  else return DC == 16 ? (((t & 3) << 1) ^ (((t >> 3) & 1) << 3)) : ((t & 3) << 1);
}

}  // namespace
}  // namespace dg
