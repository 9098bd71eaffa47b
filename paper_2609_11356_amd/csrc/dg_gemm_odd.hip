// dg_gemm_odd.hip -- the tiled pipelines on operands of any size and
// alignment: K, N, the part starts and the pointers need be no multiple of 8
// elements or 16 bytes.  Bodies, orders and bits are those of the aligned
// kernels (dg_gemm_tile.h, whose UN comment says how chunks are loaded where
// they lie and what the last slab mends); these used to run on gemm_generic,
// one wave per 16 x 16 outputs with element loads and no reuse.  Measured
// on MI355X before and after: 2047 x 14335 x 4095 16.7 ms -> 305 us (the
// aligned 2048 x 14336 x 4096: 223), 1 x 4095 x 4095 137 -> 13.5.  The sizes between the
// few-row kernels and the 256-row blocks run on the ring (dg_gemm_ring.h), as do
// tile chains and trees with fma = 1.
#include "dg_gemm_tile.h"

namespace dg {

template <int TMS, int BN, int D, int BK, bool F16>
__global__ __launch_bounds__(256) void odd_skinny(GemmArgs a) {
  skinny_body<TMS, BN, D, BK, F16, true>(a);
}

template <int BM, int BN, int WM, int WN, int BK, bool F16>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void odd_v3(GemmArgs a) {
  const int tiles_m = (int)((a.M + BM - 1) / BM);
  int ty, tx;
  grouped_tile(blockIdx.x, tiles_m, gridDim.x / tiles_m, a.order, &ty, &tx);
  v3_body<BM, BN, WM, WN, BK, F16, DG_CARRY, false, 1, true>(a, (int64_t)ty * BM, (int64_t)tx * BN);
}

template <int COMB, bool F16>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void odd_fma0(GemmArgs a) {
  const int tiles_m = (int)((a.M + 127) / 128);
  int ty, tx;
  grouped_tile(blockIdx.x, tiles_m, gridDim.x / tiles_m, a.order, &ty, &tx);
  v3_body<128, 64, 2, 2, 32, F16, COMB, true, 1, true>(a, (int64_t)ty * 128, (int64_t)tx * 64);
}

template <int BM, int BN, int BK, bool F16>
__global__ __launch_bounds__(512) void odd_pp(GemmArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t smem[2 * (BM * BK + BK * BN)];
  const int tiles_m = (int)((a.M + BM - 1) / BM);
  int ty, tx;
  grouped_tile(blockIdx.x, tiles_m, gridDim.x / tiles_m, a.order, &ty, &tx);
  pp_body<BM, BN, BK, BN, F16, true>(a, (int64_t)ty * BM, (int64_t)tx * BN, smem);
}

// ------------------------------------------------------------- launchers

template <int TMS, int BN, int D, int BK>
static hipError_t launch_skinny_o(const GemmArgs& a, hipStream_t st) {
  dim3 grid((unsigned)((a.N + BN - 1) / BN), (unsigned)((a.M + 16 * TMS - 1) / (16 * TMS)), (unsigned)a.S);
  if (a.in_f16) hipLaunchKernelGGL((odd_skinny<TMS, BN, D, BK, true>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((odd_skinny<TMS, BN, D, BK, false>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

template <int BM, int BN, int WM, int WN, int BK>
static hipError_t launch_v3_o(const GemmArgs& a, hipStream_t st) {
  const int64_t tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
  dim3 grid((unsigned)(tm * tn), 1, (unsigned)a.S);
  if (a.in_f16) hipLaunchKernelGGL((odd_v3<BM, BN, WM, WN, BK, true>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((odd_v3<BM, BN, WM, WN, BK, false>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

template <int BM, int BN, int BK>
static hipError_t launch_pp_o(const GemmArgs& a, hipStream_t st) {
  const int64_t tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
  dim3 grid((unsigned)(tm * tn), 1, (unsigned)a.S);
  if (a.in_f16) hipLaunchKernelGGL((odd_pp<BM, BN, BK, true>), grid, dim3(512), 0, st, a);
  else hipLaunchKernelGGL((odd_pp<BM, BN, BK, false>), grid, dim3(512), 0, st, a);
  return hipGetLastError();
}

template <int COMB>
static hipError_t launch_fma0_o(const GemmArgs& a, hipStream_t st) {
  const int64_t tm = (a.M + 127) / 128, tn = (a.N + 63) / 64;
  dim3 grid((unsigned)(tm * tn), 1, (unsigned)a.S);
  if (a.in_f16) hipLaunchKernelGGL((odd_fma0<COMB, true>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((odd_fma0<COMB, false>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_gemm_odd(const GemmArgs& a, int kern, int tm, int tn, hipStream_t st) {
  if (kern == 4) {
    if (tm == 16 && tn == 16) return launch_skinny_o<1, 16, 2, 256>(a, st);
    if (tm == 16 && tn == 32) return launch_skinny_o<1, 32, 2, 256>(a, st);
    if (tm == 16 && tn == 64) return launch_skinny_o<1, 64, 4, 64>(a, st);
    if (tm == 32 && tn == 64) return launch_skinny_o<2, 64, 2, 256>(a, st);
  }
  if (kern == 3) return launch_v3_o<64, 128, 2, 2, 64>(a, st);
  if (kern == 5) return launch_pp_o<256, 256, 32>(a, st);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_odd_tc(const GemmArgs& a, hipStream_t st) {
  if (a.fma != 0) return hipErrorInvalidValue;
  if (a.tile_combine == DG_CARRY) return launch_fma0_o<DG_CARRY>(a, st);
  return a.tile_combine == DG_SEQ ? launch_fma0_o<DG_SEQ>(a, st) : hipErrorInvalidValue;
}

}  // namespace dg
