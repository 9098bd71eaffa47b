// dg_gemm_ring.hip -- the ring GEMM (dg_gemm_ring.h) with a carried accumulator.
#include "dg_gemm_ring.h"

namespace dg {

template <int BM, int BN, int WM, int WN, int NS>
static hipError_t launch_ring_t(const GemmArgs& a, bool un, hipStream_t st) {
  const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const dim3 grid((unsigned)tiles, 1, (unsigned)a.S), blk(64 * WM * WN);
  if (a.in_f16 && un) hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, true, true>), grid, blk, 0, st, a);
  else if (a.in_f16) hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, true, false>), grid, blk, 0, st, a);
  else if (un) hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, false, true>), grid, blk, 0, st, a);
  else hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, false, false>), grid, blk, 0, st, a);
  return hipGetLastError();
}

hipError_t launch_gemm_ring(const GemmArgs& a, int tm, int tn, bool un, hipStream_t st) {
  if (tm == 128 && tn == 128) return launch_ring_t<128, 128, 2, 4, 4>(a, un, st);
  if (tm == 64 && tn == 128) return launch_ring_t<64, 128, 2, 4, 4>(a, un, st);
  if (tm == 64 && tn == 64) return launch_ring_t<64, 64, 2, 2, 5>(a, un, st);
  return hipErrorInvalidValue;
}

}  // namespace dg
