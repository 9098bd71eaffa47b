// dg_gemm_ring_f8.hip -- the ring GEMM (dg_gemm_ring.h) for e4m3 x e4m3.
#include "dg_gemm_ring.h"

namespace dg {

template <int BM, int BN, int WM, int WN, int NS>
static hipError_t launch_ring_f8_t(const GemmArgs& a, hipStream_t st) {
  const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, false, false, DG_CARRY, 1, 1>), dim3((unsigned)tiles, 1, (unsigned)a.S),
                     dim3(64 * WM * WN), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_gemm_ring_f8(const GemmArgs& a, int tm, int tn, hipStream_t st) {
  if (tm == 128 && tn == 128) return launch_ring_f8_t<128, 128, 2, 4, 4>(a, st);
  if (tm == 64 && tn == 128) return launch_ring_f8_t<64, 128, 2, 4, 4>(a, st);
  if (tm == 64 && tn == 64) return launch_ring_f8_t<64, 64, 2, 2, 5>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace dg
