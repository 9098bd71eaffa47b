// math_probe.hip -- test infrastructure: evaluates the library's device exp,
// SiLU and exp2 (paper_2609_11356_amd/csrc/dg_device.h, the functions of the
// fused epilogue and of the one-wave softmax and chained attention kernels)
// on a contiguous range of binary32 bit patterns, so that the tests can
// compare every binary32 input with the CPU oracle's versions; and compares
// with them the versions for non-positive inputs, which the other softmax and
// attention kernels call.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../paper_2609_11356_amd/csrc/dg_device.h"

__global__ __launch_bounds__(256) void exp_silu_range(uint64_t start, int64_t count, float* e, float* s) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
    const float x = dg::bits_f32((uint32_t)(start + (uint64_t)i));
    e[i] = dg::exp_f32(x);
    s[i] = dg::silu_f32(x);
  }
}

// e[i] = exp_f32(x), s[i] = silu_f32(x) for the binary32 value x with bits
// start + i, i < count (start + count <= 2^32); e and s are device buffers of
// count floats.  Returns a hipError_t.
extern "C" int math_probe_exp_silu(uint64_t start, int64_t count, float* e, float* s, void* stream) {
  if (count <= 0) return 0;
  if (start + (uint64_t)count > ((uint64_t)1 << 32) || !e || !s) return (int)hipErrorInvalidValue;
  int64_t blocks = (count + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(exp_silu_range, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, start, count, e, s);
  return (int)hipGetLastError();
}

__global__ __launch_bounds__(256) void exp2_range(uint64_t start, int64_t count, float* e) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256)
    e[i] = dg::exp2_f32(dg::bits_f32((uint32_t)(start + (uint64_t)i)));
}

// e[i] = exp2_f32(x) for the binary32 x with bits start + i, i < count.
extern "C" int math_probe_exp2(uint64_t start, int64_t count, float* e, void* stream) {
  if (count <= 0) return 0;
  if (start + (uint64_t)count > ((uint64_t)1 << 32) || !e) return (int)hipErrorInvalidValue;
  int64_t blocks = (count + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(exp2_range, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, start, count, e);
  return (int)hipGetLastError();
}

// bad[0], bad[1]: how many of the range's inputs, all of them non-positive or
// NaN, exp_nonpos and exp2_nonpos answer otherwise than exp_f32 and exp2_f32
// (NaNs alike); bad[2], bad[3]: the smallest such input's bits.
__global__ __launch_bounds__(256) void nonpos_range(uint64_t start, int64_t count, uint32_t* bad) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
    const uint32_t bits = (uint32_t)(start + (uint64_t)i);
    const float x = dg::bits_f32(bits);
    auto check = [&](int n, float got, float want) {
      if (dg::f32_bits(got) == dg::f32_bits(want) || (got != got && want != want)) return;
      atomicAdd(&bad[n], 1u);
      atomicMin(&bad[2 + n], bits);
    };
    check(0, dg::exp_nonpos(x), dg::exp_f32(x));
    check(1, dg::exp2_nonpos(x), dg::exp2_f32(x));
  }
}

// bad: 4 uint32 in device memory, {0, 0, ~0, ~0} before the first range.
extern "C" int math_probe_nonpos(uint64_t start, int64_t count, uint32_t* bad, void* stream) {
  if (count <= 0) return 0;
  if (start + (uint64_t)count > ((uint64_t)1 << 32) || !bad) return (int)hipErrorInvalidValue;
  int64_t blocks = (count + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(nonpos_range, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, start, count, bad);
  return (int)hipGetLastError();
}
