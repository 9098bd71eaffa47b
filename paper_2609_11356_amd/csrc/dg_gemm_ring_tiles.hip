// dg_gemm_ring_tiles.hip -- the ring GEMM (dg_gemm_ring.h) for tile chains and
// tile trees.
#include "dg_gemm_ring.h"

namespace dg {

template <int BM, int BN, int WM, int WN, int NS, int COMB, int L>
static hipError_t launch_ring_tiles_t(const GemmArgs& a, bool un, hipStream_t st) {
  const int64_t tiles = ((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN);
  const dim3 grid((unsigned)tiles, 1, (unsigned)a.S), blk(64 * WM * WN);
  if (a.in_f16 && un) hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, true, true, COMB, L>), grid, blk, 0, st, a);
  else if (a.in_f16) hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, true, false, COMB, L>), grid, blk, 0, st, a);
  else if (un) hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, false, true, COMB, L>), grid, blk, 0, st, a);
  else hipLaunchKernelGGL((gemm_ring<BM, BN, WM, WN, NS, false, false, COMB, L>), grid, blk, 0, st, a);
  return hipGetLastError();
}

hipError_t launch_gemm_ring_tiles(const GemmArgs& a, int part_tiles, int tm, int tn, bool un, hipStream_t st) {
  if (a.tile_combine == DG_SEQ) {
    if (tm == 128 && tn == 128) return launch_ring_tiles_t<128, 128, 2, 4, 4, DG_SEQ, 1>(a, un, st);
    if (tm == 64 && tn == 128) return launch_ring_tiles_t<64, 128, 2, 4, 4, DG_SEQ, 1>(a, un, st);
    if (tm == 64 && tn == 64) return launch_ring_tiles_t<64, 64, 2, 2, 5, DG_SEQ, 1>(a, un, st);
  }
  if (a.tile_combine == DG_TREE && part_tiles <= 256) {
    if (tm == 128 && tn == 128 && part_tiles <= 8) return launch_ring_tiles_t<128, 128, 2, 4, 4, DG_TREE, 3>(a, un, st);
    if (tm == 64 && tn == 128) return launch_ring_tiles_t<64, 128, 2, 4, 4, DG_TREE, 8>(a, un, st);
    if (tm == 64 && tn == 64) return launch_ring_tiles_t<64, 64, 2, 2, 5, DG_TREE, 8>(a, un, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace dg
