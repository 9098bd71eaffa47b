// dg_panel.hip -- few-row GEMMs on a packed B (the descriptor's order on a
// layout chosen for the memory system; the order, not the layout, fixes the
// bits, the point of the paper's Sec. 5.2 layout pass).
//
// A row-major B read in 16-column strips (one MFMA tile per wave, which is
// all the parallelism a few-row GEMM with one accumulator per output has)
// touches 32 bytes of every 8 KB row: measured on MI355X, 256 workgroups
// streaming such strips of a 4096 x 4096 bf16 B reach 1.5 TB/s with no
// arithmetic at all, against 4.0-4.7 TB/s for the same bytes read as
// contiguous runs.  The packed form (dg_pack_b) stores every 32 x 16 block
// of B -- 32 consecutive k of 16 consecutive columns -- as one 1 KB run in
// the operand layout of v_mfma_f32_16x16x32: lane l's 16 bytes are the 8
// values B[k0 + 8 (l / 16) + e][n0 + l % 16], e = 0..7.  Runs are ordered
// by column panel, then by k block; the panel's last columns and the last
// k block are zero-filled.
//
// gemm_panel: one wave per 16-column panel, split-K part and 16 TMS rows of
// A; each k block is one coalesced 1 KB load straight into the MFMA's B
// registers (no LDS), and A's fragment (16 bytes of one row per lane) is
// loaded beside it.  A ring of D blocks stays in flight in registers.  The
// chunks are walked in increasing k from the part start, as in every other
// kernel: a contiguous part is the blocks between its cut points (interior
// cuts on multiples of 32), a strided part the blocks of its dealt tiles
// (width a multiple of 32).  Blocks past the part's end hold zeros, whose
// chunks leave the accumulators unchanged.
//
// An e4m3 B (one byte per element) packs two k blocks per 1 KB run: lane
// l's 16 bytes are its 8 k of the first block, then its 8 k of the second,
// so each load still moves 1 KB (a 512-byte run per block measured slower
// than bf16 at one row: the loads, not the bytes, set the pace) and e4m3
// parts start on 64-k runs.  The wave widens each block's 8 values to bf16
// with the part's conversion instruction (exact) just before the bf16
// instruction, so the order and bits are those of the bf16 GEMM on the
// widened B, with half the bytes streamed.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "dg_device.h"
#include "dg_internal.h"
#include "dg_mma.h"

namespace dg {

namespace {

// A buffer offset past any record, so that it reads zero: A's bytes (below 2^31,
// the host checks) with up to 14 before its start, B's below 2^31.
constexpr uint32_t kOOB = 0x80000010u;

// 8 values of one A row from k on, each checked against K (the block that K
// cuts short, where A's rows do not lie on 16 bytes); mis: the bytes between
// the resource's start and A's.
__device__ __forceinline__ u32x4 load_a_elems(__amdgpu_buffer_rsrc_t r, uint32_t mis, int64_t row_off, int64_t k, int64_t K,
                                              bool row_ok) {
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t o0 = (row_ok && k + 2 * e < K) ? (uint32_t)((row_off + k + 2 * e) * 2) + mis : kOOB;
    const uint32_t o1 = (row_ok && k + 2 * e + 1 < K) ? (uint32_t)((row_off + k + 2 * e + 1) * 2) + mis : kOOB;
    const uint32_t lo = __builtin_amdgcn_raw_buffer_load_b16(r, o0, 0, 0);
    const uint32_t hi = __builtin_amdgcn_raw_buffer_load_b16(r, o1, 0, 0);
    w[e] = (lo & 0xffffu) | (hi << 16);
  }
  return u32x4{w[0], w[1], w[2], w[3]};
}

}  // namespace

// BT: the B operand, 0 bf16, 1 binary16 (A binary16 too), 2 OCP e4m3 bytes
// (1 KB runs of two blocks, widened to bf16 before the instruction).  The
// ring holds D runs (BPR blocks each) with the A fragments of their blocks.
// AVEC: A's rows lie on 16 bytes.  Otherwise a lane's 16 bytes are loaded where
// they lie, all but those of a last block that K cuts short, whose elements
// are loaded one by one after the ring (element loads throughout, eight a
// block and row instead of one, took 277 us at 45 x 5816 x 12713 with eight parts
// and an e4m3 B).
// FUSE: the workgroup's waves are the S <= 8 parts of one panel, and the
// partials meet in LDS in the merge's order instead of in a workspace that a
// second launch reads.
template <int TMS, int D, bool AVEC, bool STRIDED, int BT, bool FUSE>
__global__ __launch_bounds__(FUSE ? 512 : 64) void gemm_panel(GemmArgs a) {
  constexpr bool F16 = BT == 1;
  constexpr int BPR = BT == 2 ? 2 : 1;         // k blocks per 1 KB run
  constexpr int RUN = 1024;
  static_assert((D - 1) * (1 + BPR * TMS) <= 63, "the ring's waits fit the load counter");
  const int lane = threadIdx.x & 63;
  const int64_t panel = blockIdx.x;
  const int64_t i0 = (int64_t)blockIdx.y * 16 * TMS, j0 = panel * 16;
  const int s = FUSE ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : blockIdx.z;
  // every k block index fits 31 bits, every byte offset 32 (the host keeps the
  // packed B and A under 2 GiB)
  const int KR = (int)((a.K + 32 * BPR - 1) / (32 * BPR)), K = (int)a.K;
  // blocks (nf) and runs (nr) of part s: contiguous from run r0 (the host
  // puts interior cuts on run boundaries), or dealt tiles of 2^lgw blocks
  // (2^lgr runs)
  int nf = 0, r0 = 0, lgr = 0;
  if constexpr (STRIDED) {
    const int lgw = __builtin_ctz((unsigned)(a.split_w / 32));
    lgr = lgw - (BPR == 2 ? 1 : 0);
    const int w = (int)a.split_w, ntile = (K + w - 1) / w;
    nf = ntile > s ? ((ntile - s + a.S - 1) / a.S) << lgw : 0;
  } else if (a.cuts[s + 1] > a.cuts[s]) {
    r0 = (int)(a.cuts[s] / (32 * BPR));
    nf = (int)((a.cuts[s + 1] + 31) / 32) - BPR * r0;
  }
  const int nr = (nf + BPR - 1) / BPR;
  // the resource starts on 16 bytes, misA bytes before A's own start
  const uint32_t misA = AVEC ? 0 : (uint32_t)((uintptr_t)(a.A + i0 * a.K) & 15);
  const int64_t recA = (a.M - i0) * a.K * 2 + misA, recB = ((a.N + 15) / 16) * (int64_t)KR * RUN;
  const __amdgpu_buffer_rsrc_t rA = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const char*)(a.A + i0 * a.K) - misA), (short)0, (int)(uint32_t)recA, 0x00020000);
  // the panel's runs: a base moved to the panel, the run in the scalar offset
  const __amdgpu_buffer_rsrc_t rB = __builtin_amdgcn_make_buffer_rsrc((void*)a.B, (short)0, (int)recB, 0x00020000);
  const int kl = 8 * (lane >> 4);   // the lane's first k within a block
  // lane constants: B's run slot; A's row run (out of range past M), and the
  // first block whose 8 k of this lane lie at or past K (only the last block
  // when K % 32 != 0).  A block's offset goes in the scalar buffer offset.
  const uint32_t vb = (uint32_t)(panel * KR * RUN) + (uint32_t)lane * 16;
  const int flim = AVEC ? (K - kl + 31) / 32 : K / 32;
  uint32_t va[TMS];
#pragma unroll
  for (int mi = 0; mi < TMS; ++mi) {
    const int row = 16 * mi + (lane & 15);
    va[mi] = (i0 + row < a.M) ? (uint32_t)((row * K + kl) * 2) + misA : kOOB;
  }
  // runs g < nre are real (a strided part's last dealt tile may run past
  // K's last run: those runs read as zeros)
  const int nre = STRIDED ? nr : (nr < KR - r0 ? nr : KR - r0);

  // run g of the part -> global run
  auto run_of = [&](int g) -> int {
    if constexpr (STRIDED) return ((s + a.S * (g >> lgr)) << lgr) + (g & ((1 << lgr) - 1));
    else return r0 + g;
  };
  // the ring: one run of B (16 bytes per lane) and the A fragments of its blocks
  u32x4 rb[D];
  u32x4 ra[D][BPR][TMS];
  auto load = [&](int u, int g) {
    const int R = run_of(g);
    const bool ok = g < nre && (!STRIDED || R < KR);
    const int so = ok ? R : 0;
    rb[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rB, ok ? vb : kOOB, so * RUN, 0));
#pragma unroll
    for (int h = 0; h < BPR; ++h) {
      const int f = BPR * so + h;
#pragma unroll
      for (int mi = 0; mi < TMS; ++mi)
        ra[u][h][mi] = __builtin_bit_cast(
            u32x4, __builtin_amdgcn_raw_buffer_load_b128(rA, (ok && f < flim) ? va[mi] : kOOB, f * 64, 0));
    }
  };

  floatx4 acc[TMS];
#pragma unroll
  for (int mi = 0; mi < TMS; ++mi) acc[mi] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto products = [&](const u32x4& b, int h, const u32x4* fa) {
    u32x4 bw;
    if constexpr (BT == 2)
      bw = u32x4{e4m3x2_bf16x2<false>(b[2 * h]), e4m3x2_bf16x2<true>(b[2 * h]), e4m3x2_bf16x2<false>(b[2 * h + 1]),
                 e4m3x2_bf16x2<true>(b[2 * h + 1])};
    else
      bw = b;
#pragma unroll
    for (int mi = 0; mi < TMS; ++mi)
      acc[mi] = mfma16t<F16>(__builtin_bit_cast(shortx8, fa[mi]), __builtin_bit_cast(shortx8, bw), acc[mi]);
  };
  // The loads stay in ring order (no scheduling across the barriers): the
  // waits count on run g's loads being older than those of g + 1.
  static_for<0, D>([&](auto u) {
    load(u, u);
    __builtin_amdgcn_sched_barrier(0);
  });
  for (int base = 0; base < nr; base += D) {
    static_for<0, D>([&](auto u) {
      const int g = base + u;
      // this run's loads are the oldest of D groups in flight
      __builtin_amdgcn_s_waitcnt(vmcnt_only((D - 1) * (1 + BPR * TMS)));
#pragma unroll
      for (int h = 0; h < BPR; ++h)
        if (BPR * g + h < nf && (AVEC || BPR * run_of(g) + h < flim)) products(rb[u], h, ra[u][h]);
      load(u, g + D);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  if constexpr (!AVEC) {
    // the block that K cuts short, the last of the part that holds it
    const int f = K / 32;
    bool mine = K % 32 != 0;
    if constexpr (STRIDED) mine = mine && (f * 32 / (int)a.split_w) % a.S == s;
    else mine = mine && f >= BPR * r0 && f < BPR * r0 + nf;
    if (mine) {
      const u32x4 b = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rB, vb, f / BPR * RUN, 0));
      u32x4 fa[TMS];
#pragma unroll
      for (int mi = 0; mi < TMS; ++mi) {
        const int row = 16 * mi + (lane & 15);
        fa[mi] = load_a_elems(rA, misA, (int64_t)row * a.K, (int64_t)f * 32 + kl, a.K, i0 + row < a.M);
      }
      if (BPR == 2 && (f & 1)) products(b, BPR - 1, fa);
      else products(b, 0, fa);
    }
  }
  if constexpr (!FUSE) {
#pragma unroll
    for (int mi = 0; mi < TMS; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + 16 * mi + 4 * (lane >> 4) + r, j = j0 + (lane & 15);
        if (i < a.M && j < a.N) finish(a, s, i, j, acc[mi][r]);
      }
  } else {
    __shared__ float part[8][16 * TMS][16];
#pragma unroll
    for (int mi = 0; mi < TMS; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        part[s][16 * mi + 4 * (lane >> 4) + r][lane & 15] = a.partial_bf16 ? round_bf16(acc[mi][r]) : acc[mi][r];
    __syncthreads();
    GemmArgs b = a;   // finish as a single part would, the partials rounded already
    b.S = 1;
    b.partial_bf16 = 0;
    auto add = [&](float x, float y) {
      const float v = x + y;
      return a.merge_bf16 ? round_bf16(v) : v;
    };
    for (int q = threadIdx.x; q < 16 * TMS * 16; q += blockDim.x) {
      const int row = q / 16, col = q % 16;
      if (i0 + row >= a.M || j0 + col >= a.N) continue;
      float y = 0.f;
      if (a.split_combine == DG_SEQ) {
        y = part[0][row][col];
        for (int t = 1; t < a.S; ++t) y = add(y, part[t][row][col]);
      } else {
        // balanced tree: a binary counter's levels, folded low to high
        float l0 = 0.f, l1 = 0.f, l2 = 0.f, l3 = 0.f;
        for (int t = 0; t < a.S; ++t) {
          float v = part[t][row][col];
          if (!(t & 1)) { l0 = v; continue; }
          v = add(l0, v);
          if (!(t & 2)) { l1 = v; continue; }
          v = add(l1, v);
          if (!(t & 4)) { l2 = v; continue; }
          l3 = add(l2, v);
        }
        bool have = false;
        auto meet = [&](int lv, float x) {
          if (!((a.S >> lv) & 1)) return;
          y = have ? add(x, y) : x;
          have = true;
        };
        meet(0, l0);
        meet(1, l1);
        meet(2, l2);
        meet(3, l3);
      }
      finish(b, 0, i0 + row, j0 + col, y);
    }
  }
}

// The packed form of B (K x N, 16-bit elements, row-major): thread t writes
// lane l = t % 64 of run t / 64 (panel p = run / KB, k block f = run % KB).
__global__ __launch_bounds__(256) void pack_b(const uint16_t* __restrict__ B, uint16_t* __restrict__ Bp, int64_t K,
                                              int64_t N, int64_t runs) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= runs * 64) return;
  const int64_t run = t / 64, KB = (K + 31) / 32;
  const int l = (int)(t % 64);
  const int64_t p = run / KB, f = run % KB;
  const int64_t n = p * 16 + (l & 15), k0 = f * 32 + 8 * (l >> 4);
  uint32_t w[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t lo = (n < N && k0 + 2 * e < K) ? B[(k0 + 2 * e) * N + n] : 0;
    const uint32_t hi = (n < N && k0 + 2 * e + 1 < K) ? B[(k0 + 2 * e + 1) * N + n] : 0;
    w[e] = lo | (hi << 16);
  }
  *(u32x4*)&Bp[t * 8] = u32x4{w[0], w[1], w[2], w[3]};
}

// One-byte elements: every 64 x 16 block (two k blocks) is one 1 KB run, lane
// l's 16 bytes holding its 8 k of the first block, then its 8 k of the
// second: thread t writes lane l = t % 64 of run t / 64 (panel p = run / KR,
// run r = run % KR of the panel).
__global__ __launch_bounds__(256) void pack_b8(const uint8_t* __restrict__ B, uint8_t* __restrict__ Bp, int64_t K,
                                               int64_t N, int64_t runs) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= runs * 64) return;
  const int64_t run = t / 64, KR = (K + 63) / 64;
  const int l = (int)(t % 64);
  const int64_t p = run / KR, r = run % KR;
  const int64_t n = p * 16 + (l & 15), k0 = r * 64 + 8 * (l >> 4);
  uint32_t w[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    uint32_t v = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t k = k0 + 32 * (q >> 1) + 4 * (q & 1) + e;
      v |= (uint32_t)((n < N && k < K) ? B[k * N + n] : 0) << (8 * e);
    }
    w[q] = v;
  }
  *(u32x4*)&Bp[t * 16] = u32x4{w[0], w[1], w[2], w[3]};
}

hipError_t launch_pack_b8(const uint8_t* B, uint8_t* Bp, int64_t K, int64_t N, hipStream_t st) {
  const int64_t runs = ((N + 15) / 16) * ((K + 63) / 64);
  const int64_t blocks = (runs * 64 + 255) / 256;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(pack_b8, dim3((unsigned)blocks), dim3(256), 0, st, B, Bp, K, N, runs);
  return hipGetLastError();
}

hipError_t launch_pack_b(const uint16_t* B, uint16_t* Bp, int64_t K, int64_t N, hipStream_t st) {
  const int64_t runs = ((N + 15) / 16) * ((K + 31) / 32);
  const int64_t blocks = (runs * 64 + 255) / 256;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(pack_b, dim3((unsigned)blocks), dim3(256), 0, st, B, Bp, K, N, runs);
  return hipGetLastError();
}

// an e4m3 ring of D runs holds 2 D TMS A fragments (16 bytes per lane each),
// and its waits count up to (D - 1)(1 + 2 TMS) loads (the counter holds 63)
constexpr bool panel_b8_fits(int tms, int d) { return 2 * d * tms <= 48 && (d - 1) * (1 + 2 * tms) <= 63; }

// Ring depths measured best on MI355X (4096 x 4096 B, M = 1, 7, 32, 64);
// an e4m3 ring's runs hold two blocks each
constexpr int default_depth(int tms, bool b8) {
  if (b8) return tms == 4 ? 6 : 8;
  return tms == 4 ? 10 : 16;
}
int panel_default_depth(int tms, bool b8) { return default_depth(tms, b8); }

// The parts meet inside the kernel where they are two to eight contiguous
// ones, at the library's own depth: no partials, no second launch (8 x 4096 x
// 14336 in eight parts 29.6 -> 23.9 us, 1 x 1024 x 1024 in two 11.9 -> 6.3). A
// workgroup then reads on one CU what its parts read on f where panels are few
// (16 x 512 x 8192 in eight parts 11.75 us apart, 12.75 merged; 64 x 512 x
// 14336 16.3 and 58; 64 x 1024 x 2048 in four 9.9 and 13.2; 48 x 3072 x 4096
// in three, f = 1.3, 22.3 and 19.6), so it must not be more than the second
// launch saves: the share that others would read, squared, of some 155 KB with
// 16 rows a wave, 77 with 32, 53 with 64.  Where panels are more than the CUs,
// S waves that end together fill the last round worse than S waves of their
// own, by the empty part of the round and about a tenth (up to 8 rows, which
// wait for HBM, 3 %), which grows with K while what merging saves (the launch,
// the partials written and read) does not: 64 x 5760 x 14336 in two parts 97.4
// us apart, 128 merged; 64 x 5760 x 512 12.6 and 11.2; 64 x 8192 x 14336 in
// eight 136 and 143, x 2048 41.0 and 30.1.  With the panels' bytes at 16 TB/s
// (20 up to 8 rows; A's come from the caches) and the partials' at 4.2, the
// estimate below takes the faster way, or one within 7 % of it, at 98 % of
// 4164 measured sizes (operands from HBM).
bool panel_merges(const GemmArgs& a, int tms, int depth, int ncu) {
  const bool b8 = a.b_e4m3 != 0;
  if (a.S < 2 || a.S > 8 || a.split_w != 0 || depth != default_depth(tms, b8)) return false;
  const double panels = (double)((a.N + 15) / 16) * (double)((a.M + 16 * tms - 1) / (16 * tms));
  const double rows = std::min<double>(a.M, 16 * tms) / 16, runs = (double)a.K / (b8 ? 64 : 32);
  const double kb = runs * (1 + (b8 ? 2 : 1) * rows);   // KB of B and A that a panel's parts read
  if (panels < ncu) {
    const double apart = 1 - 1 / std::min<double>(a.S, ncu / panels);   // the share that other CUs would read
    return kb * apart * apart <= (tms == 1 ? 155 : tms == 2 ? 77 : 53) && runs * (1 + (b8 ? 2 : 1) * tms) * apart <= 250;
  }
  const double rounds = std::ceil(panels / ncu);
  const double empty = rounds * ncu / panels - 1 + (panels > ncu ? (a.M <= 8 ? 0.03 : 0.11) : 0);
  return panels * kb * empty / (a.M <= 8 ? 20000 : 16000) <= 2.5 + 8.0 * a.S * (double)a.M * (double)a.N / 4.2e6;   // us
}

template <int TMS, int D, bool AVEC>
static hipError_t launch_panel_t(const GemmArgs& a, bool merge, hipStream_t st) {
  const unsigned panels = (unsigned)((a.N + 15) / 16), rows = (unsigned)((a.M + 16 * TMS - 1) / (16 * TMS));
  const bool strided = a.split_w != 0;
  const int bt = a.b_e4m3 ? 2 : a.in_f16 ? 1 : 0;
  auto go = [&](auto BT_) {
    constexpr int BT = decltype(BT_)::value;
    const dim3 grid(panels, rows, (unsigned)a.S);
    if (strided) hipLaunchKernelGGL((gemm_panel<TMS, D, AVEC, true, BT, false>), grid, dim3(64), 0, st, a);
    else if (merge) {   // panel_merges: at the default depth
      if constexpr (D == default_depth(TMS, BT == 2))
        hipLaunchKernelGGL((gemm_panel<TMS, D, AVEC, false, BT, true>), dim3(panels, rows), dim3(64 * a.S), 0, st, a);
    }
    else hipLaunchKernelGGL((gemm_panel<TMS, D, AVEC, false, BT, false>), grid, dim3(64), 0, st, a);
  };
  if (bt == 2) {
    // two blocks per run: the rings whose A fragments fit the registers
    if constexpr (panel_b8_fits(TMS, D)) go(std::integral_constant<int, 2>{});
    else return hipErrorInvalidValue;
  }
  else if (bt == 1) go(std::integral_constant<int, 1>{});
  else go(std::integral_constant<int, 0>{});
  return hipGetLastError();
}

// (rows of A per wave / 16, ring depth) pairs built, for 16-byte A runs and
// for any other A
#define DG_PANEL_LIST(X) \
  X(1, 8) X(1, 16) X(1, 24) X(1, 32) X(2, 8) X(2, 12) X(2, 16) X(4, 6) X(4, 10)
#define DG_PANEL_ANY_LIST(X) X(1, 8) X(1, 16) X(2, 8) X(2, 16) X(4, 6) X(4, 10)

bool panel_supported(int tms, int depth, bool b8) {
  if (b8 && !panel_b8_fits(tms, depth)) return false;
#define DG_PANEL_HAS(T_, D_) \
  if (tms == T_ && depth == D_) return true;
  DG_PANEL_LIST(DG_PANEL_HAS)
#undef DG_PANEL_HAS
  return false;
}

hipError_t launch_gemm_panel(const GemmArgs& a, int tms, int depth, bool avec, bool merge, hipStream_t st) {
#define DG_PANEL_RUN(T_, D_) \
  if (tms == T_ && depth == D_) return launch_panel_t<T_, D_, AVEC_>(a, merge, st);
  if (avec) {
    constexpr bool AVEC_ = true;
    DG_PANEL_LIST(DG_PANEL_RUN)
  } else {
    constexpr bool AVEC_ = false;
    DG_PANEL_ANY_LIST(DG_PANEL_RUN)
  }
#undef DG_PANEL_RUN
  return hipErrorInvalidValue;
}

}  // namespace dg
