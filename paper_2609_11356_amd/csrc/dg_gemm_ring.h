// dg_gemm_ring.h -- bf16 / binary16 / e4m3 GEMM on BM x BN blocks with a ring of
// NS LDS slots filled by direct-to-LDS loads, for the sizes between the
// few-row kernels and the 256-row blocks: the order and bits of the other
// chunk-grid kernels (8-k chunks in increasing k through one accumulator, on
// the 32x32x16 instruction).
//
// Bound: latency on short grids, LDS and the load path on full ones.  The v3
// kernel (two slabs ahead through registers, LDS writes, a barrier between)
// took 1150 cycles per 64-k slab of a 64 x 128 block however few MFMAs it
// held; the ping-pong kernel 1400 per slab of 128 x 128 (512 of MFMA).  Here
// a slab's loads have no register or LDS-write stage, three slabs (of four
// slots) or four (of five) are in flight, and the wave reads the next 16-k
// step's fragments while it issues the MFMAs of this one.  One barrier per slab, before its last step:
//   wait until the wave's own loads of slab s + 1 have landed, barrier; then
//   the fragments of slab s + 1 may be read (every wave's loads of it are
//   in), and the slot of slab s - 1 may be filled again (every wave has
//   issued its MFMAs of slab s - 1): its NI loads, for slab s + NS - 1, are
//   spread over the next four steps.
// Slabs past the part end are zeros (their chunks leave accumulators as they
// are).  A [row][k], 128-byte rows, chunk c of row r at c ^ ((r / 2) mod 8):
// 16 consecutive rows of one chunk on 16 slots of a 256-byte bank window.
// B [k][n]: 64 bytes of 4 k rows per half wave of a transposing read, on 16
// slots.
// Measured on MI355X before and after (v3, ping-pong and few-row kernels):
// 1024 x 4096 x 4096 44.5 -> 37.0 us, 512 x 4096 x 4096 39 -> 24.6, 256 x 4096
// x 4096 38 -> 17.9, 1024 x 1024 x 1024 13.5 -> 7.3, 128 x 14336 x 4096 89 ->
// 25.6, 32 x 14336 x 4096 36.8 -> 21.9, 1 x 14272 x 3328 54 -> 16; odd sizes
// 515 x 3001 x 2047 33 -> 21.  Blocks of 128 x 128 with 2 x 4 waves beat 2 x 2
// (37 against 42 us) and 4 x 2 (39); the 64 x 128 ones 2 x 2 (24.6 against
// 26).  64 x 64: five slots (80 KB, two blocks fit a CU) 17.5, six 17.9, four
// 19.7.
// Tile chains and trees (COMB): a wave's block is one 32-row accumulator of
// 16 or 32 registers, so an eight-level stack of closed tiles (256 of them) fits beside it.
// tile_k 64 trees, before (gemm_tc: 128-row blocks, so that most sizes filled a
// few CUs) and after: 256 x 4096 x 4096 70.8 -> 27.8 us, 1024 x 4096 x 4096 140
// -> 62, 2048 x 14336 x 4096 963 -> 510, 1 x 1024 x 1024 18.9 -> 10.1.
// EB = 1, e4m3 (128-k slabs of the same bytes, two 64-k steps): before (kernel
// 13's 256 x 128 blocks) and after 256 x 4096 x 4096 34.6 -> 14.2 us, 1024 x 4096
// x 4096 35.3 -> 21.7, 16 x 4096 x 14336 101 -> 35, 64 x 14336 x 4096 34.8 -> 15.3.
// B's transposing reads take 8 rows x 32 columns per half wave, whose 16
// chunks the swizzle puts on 16 slots.
// UN (odd sizes): chunks are loaded where they lie, as in dg_gemm_tile.h, and
// the lanes that loaded the last slab mend it in LDS before it is read.
#pragma once

#include "dg_gemm_tile.h"

namespace dg {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void* lds_void;
typedef int intx2 __attribute__((ext_vector_type(2)));
typedef int intx8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) intx2* lds_i2;

// LDS array number ID of the workgroup (one per slot, A's slab and then B's, so
// that the compiler can tell a read of one slot from the loads in flight to
// the others).
template <int ID, int BYTES>
__device__ __forceinline__ uint16_t* ring_array() {
  __shared__ __attribute__((aligned(1024))) uint16_t L[BYTES / 2];
  return L;
}

__device__ __forceinline__ void ring_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <bool F16>
__device__ __forceinline__ void mfma32(floatx16& c, const shortx8& a, const shortx8& b) {
  if constexpr (F16)
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  else
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

}  // namespace

template <int BM, int BN, int WM, int WN, int NS, bool F16, bool UN, int COMB = DG_CARRY, int L = 1, int EB = 2>
__global__ __launch_bounds__(64 * WM * WN) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_ring(GemmArgs a) {
  // EB: bytes per element; a slab is 128 bytes of k, a step one MFMA of k
  constexpr int NW = WM * WN, BK = 128 / EB, EPC = 16 / EB, STEPS = EB == 2 ? 4 : 2, WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int BROW = BN / EPC, A_BYTES = BM * 128, B_BYTES = BK * BN * EB;
  constexpr int NIA = A_BYTES / 1024 / NW, NIB = B_BYTES / 1024 / NW, NI = NIA + NIB;   // loads per wave and slab
  static_assert(A_BYTES % (1024 * NW) == 0 && B_BYTES % (1024 * NW) == 0 && TM >= 1 && TN >= 1, "whole loads and tiles");
  static_assert((BROW == 4 || BROW == 8 || BROW == 16) && (EB == 2 || (!UN && COMB == DG_CARRY)) && NS >= 4 && NS <= 6 && (NS - 1) * NI <= 63, "the waits fit the load counter");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int tiles_m = (int)((a.M + BM - 1) / BM);
  int ty, tx;
  grouped_tile(blockIdx.x, tiles_m, gridDim.x / tiles_m, a.order, &ty, &tx);
  const int64_t i0 = (int64_t)ty * BM, j0 = (int64_t)tx * BN;
  const int s = blockIdx.z;
  const int64_t k0 = a.cuts[s], k1 = a.cuts[s + 1];
  const int nslab = (int)((k1 - k0 + BK - 1) / BK);
  auto swA = [](int r) { return (r >> 1) & 7; };
  auto swB = [](int k) {
    if constexpr (EB == 1) return BROW == 8 ? ((k >> 1) & 3) << 1 : ((k >> 2) & 1) << 1;
    else return BROW == 16 ? (k & 3) << 2 : ((k >> 1) & 1) << 2;
  };

  // load t of the wave fills 1 KB: A rows 8 (NIA wave + t).., or B rows; each
  // lane fetches the chunk that belongs at its place (a row past M or a
  // column past N lies past the resource's end and reads zero)
  constexpr uint32_t OOB = 0x80000000u;
  constexpr int BRUN = 64 / BROW;               // B rows per load
  // place of the lane's chunk of load t: A row and first k, B k row and first column
  auto place_a = [&](int t, int* row, int* k) { *row = (NIA * wave + t) * 8 + lane / 8; *k = EPC * ((lane & 7) ^ swA(*row)); };
  auto place_b = [&](int u, int* kr, int* col) {
    *kr = (NIB * wave + u) * BRUN + lane / BROW;
    *col = EPC * ((lane % BROW) ^ swB(*kr));
  };
  // UN: the resources start on 16 bytes, mis* bytes before the operands' own start
  const char *pA = (const char*)a.A + i0 * a.K * EB, *pB = (const char*)a.B + k0 * a.N * EB;
  const uint32_t misA = UN ? (uint32_t)((uintptr_t)pA & 15) : 0, misB = UN ? (uint32_t)((uintptr_t)pB & 15) : 0;
  uint32_t off[NI];
  int kl[NI];   // the chunk is loaded while this k lies before the part end
#pragma unroll
  for (int t = 0; t < NIA; ++t) {
    int row, k;
    place_a(t, &row, &k);
    off[t] = i0 + row < a.M ? (uint32_t)((row * a.K + k) * EB) + misA : OOB;
    kl[t] = UN && k1 == a.K && i0 + row == a.M - 1 ? k + 7 : k;             // the matrix's last chunk only whole
  }
#pragma unroll
  for (int u = 0; u < NIB; ++u) {
    int kr, col;
    place_b(u, &kr, &col);
    off[NIA + u] = j0 + col < a.N ? (uint32_t)((kr * a.N + j0 + col) * EB) + misB : OOB;
    kl[NIA + u] = UN && k1 == a.K && j0 + col + 8 > a.N ? kr + 1 : kr;
  }
  const int64_t recA = (a.M - i0) * a.K * EB + misA, recB = (a.K - k0) * a.N * EB + misB;
  const __amdgpu_buffer_rsrc_t rA = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(pA - misA), (short)0, (int)(recA < 0x7fffffff ? recA : 0x7fffffff), 0x00020000);
  const __amdgpu_buffer_rsrc_t rB = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(pB - misB), (short)0, (int)(recB < 0x7fffffff ? recB : 0x7fffffff), 0x00020000);
  const int stepB = (int)(BK * a.N * EB);
  // load t of slab sl into slot X
  auto dma = [&](int sl, auto X, auto T) {
    constexpr int x = decltype(X)::value, t = decltype(T)::value;
    const int left = sl < nslab ? (int)(k1 - k0) - sl * BK : 0;   // k of the part from the slab on
    const uint32_t o = kl[t] < left ? off[t] : OOB;
    if constexpr (t < NIA)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rA, (lds_void)(ring_array<x, A_BYTES + B_BYTES>() + 512 * (NIA * wave + t)), 16, o,
                                               sl < nslab ? (int)((k0 + sl * BK) * EB) : 0, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rB, (lds_void)(ring_array<x, A_BYTES + B_BYTES>() + A_BYTES / 2 + 512 * (NIB * wave + t - NIA)), 16, o, sl < nslab ? sl * stepB : 0, 0, 0);
  };

  // UN: the part's last slab, in slot X, is mended by the lanes that loaded
  // it: elements of A at or past the part end are cleared, and the chunk that
  // ends each matrix is put together from single elements.
  auto mend = [&](auto X) {
    uint16_t* base = ring_array<decltype(X)::value, A_BYTES + B_BYTES>() + 8 * lane;
    const int64_t kb = k0 + (int64_t)(nslab - 1) * BK;
    static_for<0, NIA>([&](auto T) {
      int row, k;
      place_a(decltype(T)::value, &row, &k);
      u32x4* p = (u32x4*)(base + 512 * (NIA * wave + decltype(T)::value));
      if (i0 + row < a.M && kb + k < k1 && kb + k + 8 > k1) *p = last_a(a, *p, i0 + row, kb + k, k1);
    });
    static_for<0, NIB>([&](auto T) {
      int kr, col;
      place_b(decltype(T)::value, &kr, &col);
      u32x4* p = (u32x4*)(base + A_BYTES / 2 + 512 * (NIB * wave + decltype(T)::value));
      if (kb + kr == a.K - 1 && j0 + col < a.N && j0 + col + 8 > a.N) *p = last_b(a, *p, kb + kr, j0 + col, k1);
    });
    lds_wait();
  };

  floatx16 acc[TM][TN];
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
  // tile combine: acc is the open tile; the chain's running sum or the tree's
  // stack (a binary counter's levels) holds the closed ones
  constexpr int NL = COMB == DG_TREE ? L : COMB == DG_SEQ ? 1 : 0;
  floatx16 stk[NL > 0 ? NL : 1][TM][TN];
  uint32_t count = 0;                                  // tiles closed
  const int len = (int)(k1 - k0), tk = (int)(a.tile_k < len ? a.tile_k : len);
  int tile_end = a.tail_first && tk > 0 && len % tk ? len % tk : tk;   // of the open tile, from the part start
  auto each = [&](auto f) {
    static_for<0, TM>([&](auto mi) { static_for<0, TN>([&](auto ni) { f(mi, ni); }); });
  };
  auto close_tile = [&]() {
    const bool last = tile_end >= len;
    if constexpr (COMB == DG_SEQ) {
      if (count == 0) each([&](auto mi, auto ni) { stk[0][mi][ni] = acc[mi][ni]; });
      else each([&](auto mi, auto ni) { stk[0][mi][ni] = stk[0][mi][ni] + acc[mi][ni]; });
    } else if constexpr (COMB == DG_TREE) {
      // fold the levels whose bit is set, park at the first clear one (the
      // last tile's value needs no parking: it stays in acc)
      bool parked = false;
      static_for<0, NL>([&](auto lv) {
        constexpr int LV = decltype(lv)::value;
        if (!parked) {
          if ((count >> LV) & 1u) each([&](auto mi, auto ni) { acc[mi][ni] = stk[LV][mi][ni] + acc[mi][ni]; });
          else {
            each([&](auto mi, auto ni) { stk[LV][mi][ni] = acc[mi][ni]; });
            parked = true;
          }
        }
      });
    }
    ++count;
    if (COMB == DG_SEQ || !last)
      each([&](auto mi, auto ni) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
      });
    tile_end = last ? 0x7fffffff : tile_end + tk < len ? tile_end + tk : len;
  };
  typedef std::conditional_t<EB == 2, shortx8, intx8> Frag;
  Frag fa[2][TM], fb[2][TN];
  // the lane's addresses within the slabs, in bytes (the A chunk moves under
  // its swizzle, the B rows by a constant)
  const int ar = wm * WTM + (lane & 31), h = lane >> 5;
  const int vi = lane & 15, br = EB == 2 ? 8 * h + (vi >> 2) : 16 * h + (vi >> 1);
  const int bc = wn * WTN + 16 * ((lane >> 4) & 1) + (EB == 2 ? 4 * (vi & 3) : 8 * (vi & 1));
  int ad[4], bd[TN];
#pragma unroll
  for (int j = 0; j < 4; ++j) ad[j] = ar * 128 + 16 * ((2 * j + h) ^ swA(ar));
#pragma unroll
  for (int ni = 0; ni < TN; ++ni) {
    const int c = bc + 32 * ni;
    bd[ni] = EB * br * BN + 16 * ((c / EPC) ^ swB(br)) + EB * (c % EPC);
  }
  // fragments of step j of the slab in slot X, into set x
  auto read = [&](auto X, int j, int x) {
    const char* As = (const char*)ring_array<decltype(X)::value, A_BYTES + B_BYTES>();
    const char* Bs = As + A_BYTES;
    if constexpr (EB == 2) {
#pragma unroll
      for (int mi = 0; mi < TM; ++mi) fa[x][mi] = *(const shortx8*)&As[ad[j] + 32 * mi * 128];
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&Bs[bd[ni] + 16 * j * BN * 2]));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&Bs[bd[ni] + (16 * j + 4) * BN * 2]));
        fb[x][ni] = shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      }
    } else {
      // a lane's 32 bytes: k = 16h + 0..15 and 32 + 16h + 0..15 of the step's 64
#pragma unroll
      for (int mi = 0; mi < TM; ++mi) {
        const u32x4 lo = *(const u32x4*)&As[ad[2 * j] + 32 * mi * 128];
        const u32x4 hi = *(const u32x4*)&As[ad[2 * j + 1] + 32 * mi * 128];
        fa[x][mi] = intx8{(int)lo[0], (int)lo[1], (int)lo[2], (int)lo[3], (int)hi[0], (int)hi[1], (int)hi[2], (int)hi[3]};
      }
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        intx2 v[4];
#pragma unroll
        for (int p = 0; p < 4; ++p)
          v[p] = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i2)(&Bs[bd[ni] + (64 * j + 8 * (p & 1) + 32 * (p >> 1)) * BN]));
        fb[x][ni] = intx8{v[0][0], v[0][1], v[1][0], v[1][1], v[2][0], v[2][1], v[3][0], v[3][1]};
      }
    }
  };
  auto products = [&](int x) {
#pragma unroll
    for (int mi = 0; mi < TM; ++mi)
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        if constexpr (EB == 2) mfma32<F16>(acc[mi][ni], fa[x][mi], fb[x][ni]);
        else   // the block-scaled instruction with unit scales: the chain of 16-k chunks
          acc[mi][ni] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fa[x][mi], fb[x][ni], acc[mi][ni], 0, 0, 0, 127, 0, 127);
      }
  };

  // prologue: slabs 0 .. NS - 2 on their way, slab 0 in, its first fragments read
  static_for<0, NS - 1>([&](auto x) { static_for<0, NI>([&](auto t) { dma(x, x, t); }); });
  __builtin_amdgcn_s_waitcnt(vmcnt_only((NS - 2) * NI));
  if constexpr (UN)
    if (nslab == 1) mend(std::integral_constant<int, 0>{});
  ring_barrier();
  read(std::integral_constant<int, 0>{}, 0, 0);
  // the loads owed to the slot freed by the last barrier: slab `next`, slot
  // (x + NS - 1) % NS, a share per step
  auto slab = [&](int sl, auto X, auto MEND) {   // MEND: slab sl + 1 may be the last
    constexpr int x = decltype(X)::value;
    constexpr std::integral_constant<int, (x + 1) % NS> nxt{};
    constexpr std::integral_constant<int, (x + NS - 1) % NS> prev{};   // slot of slab sl - 1: takes slab sl + NS - 1
    constexpr std::integral_constant<int, (x + 2 * NS - 2) % NS> old{};  // slot of slab sl - 2: takes slab sl + NS - 2
    static_for<0, STEPS>([&](auto J) {
      constexpr int j = decltype(J)::value;
      if constexpr (j == STEPS - 1) {
        // own loads of slab sl + 1 in (slabs sl + 2 .. sl + NS - 2 may be out), then everybody's
        __builtin_amdgcn_s_waitcnt(vmcnt_only((NS - 3) * NI));
        if constexpr (UN && decltype(MEND)::value)
          if (sl + 2 == nslab) mend(nxt);
        ring_barrier();
        read(nxt, 0, 0);
      } else {
        read(X, j + 1, (j + 1) & 1);
      }
      products(j & 1);
      if constexpr (COMB != DG_CARRY && (j & 1))   // every tile ends on a 32-k step, or the part does
        if (64 * sl + 16 * j + 16 >= tile_end) close_tile();
      // the last step begins the loads of slab sl + NS - 1; the others finish those
      // that the slab before began (the first slab has none to finish)
      static_for<0, NI>([&](auto T) {
        constexpr int t = decltype(T)::value, q = t * STEPS / NI;   // the first with this slab's last step
        if constexpr (j == STEPS - 1) {
          if constexpr (q == 0) dma(sl + NS - 1, prev, T);
        } else if constexpr (q == j + 1) {
          if (sl > 0) dma(sl + NS - 2, old, T);
        }
      });
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  int sl = 0;   // the loop leaves 1 to NS slabs: the last one is in the rest
  for (; sl + NS < nslab; sl += NS)
    static_for<0, NS>([&](auto x) { slab(sl + x, x, std::integral_constant<bool, decltype(x)::value == NS - 1>{}); });
  static_for<0, NS>([&](auto x) {
    if (sl + decltype(x)::value < nslab) slab(sl + decltype(x)::value, x, std::integral_constant<bool, decltype(x)::value != NS - 1>{});
  });
  // the part's value: the chain's sum, or the tree's stack folded low to high
  // (acc holds the entry of level ctz(count); the set levels above meet it)
  // (an empty part, K = 0, has closed no tile: acc is its value)
  if constexpr (COMB == DG_SEQ)
    if (count) each([&](auto mi, auto ni) { acc[mi][ni] = stk[0][mi][ni]; });
  if constexpr (COMB == DG_TREE) {
    const int low = count ? __builtin_ctz(count) : 0;
    static_for<0, NL>([&](auto lv) {
      constexpr int LV = decltype(lv)::value;
      if (LV > low && ((count >> LV) & 1u)) each([&](auto mi, auto ni) { acc[mi][ni] = stk[LV][mi][ni] + acc[mi][ni]; });
    });
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));   // nothing lands in the staging area later
  __syncthreads();

  // epilogue: the block's bias as binary32 in slot 0's B array; each wave
  // stages 16-row halves of its bands through its part of the A arrays
  // (pitch WTN + 8 floats: the two row sets of one write 32 banks apart) and
  // finishes four columns per store
  constexpr int CSP = WTN + 8, CSB = 16 * CSP * 4, PER = A_BYTES / CSB;
  static_assert(PER >= 1 && PER * NS >= NW && BN * 4 <= B_BYTES, "epilogue staging fits");
  float* bsh = reinterpret_cast<float*>(ring_array<0, A_BYTES + B_BYTES>() + A_BYTES / 2);
  stage_bias(a, j0, BN, bsh);
  __syncthreads();
  const bool bias = needs_bias(a);
  float* cs = nullptr;
  static_for<0, NS>([&](auto x) {
    if (wave / PER == decltype(x)::value)
      cs = reinterpret_cast<float*>(ring_array<decltype(x)::value, A_BYTES + B_BYTES>()) + (wave % PER) * 16 * CSP;
  });
#pragma unroll
  for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
#pragma unroll
      for (int ni = 0; ni < TN; ++ni)
#pragma unroll
        for (int r = 8 * half; r < 8 * half + 8; ++r)
          cs[(8 * (r / 4) - 16 * half + 4 * h + (r & 3)) * CSP + 32 * ni + (lane & 31)] = acc[mi][ni][r];
      lds_wait();
#pragma unroll 2
      for (int q = lane; q < 16 * WTN / 4; q += 64) {
        const int rr = q / (WTN / 4), cc = 4 * (q % (WTN / 4));
        const int64_t gi = i0 + wm * WTM + 32 * mi + 16 * half + rr, gj = j0 + wn * WTN + cc;
        const float4 b4 = bias ? *(const float4*)&bsh[wn * WTN + cc] : float4{0.f, 0.f, 0.f, 0.f};
        if (gi < a.M && gj < a.N) (void)finish4v<UN>(a, s, gi, gj, *(const float4*)&cs[rr * CSP + cc], b4);
      }
      lds_wait();
    }
  }
}

}  // namespace dg
