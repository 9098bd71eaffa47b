// dg_gemm_tile.h -- the tiled GEMM pipelines shared by the aligned kernels
// (dg_gemm.hip) and the odd-sized ones (dg_gemm_odd.hip): operand chunks, the
// output finish, the block orders, and the bodies of the transposing-read
// (v3), ping-pong (pp) and few-row (skinny) kernels.
#pragma once

#include <type_traits>

#include "dg_device.h"
#include "dg_internal.h"
#include "dg_mma.h"

namespace dg {

// Sixteen zero bytes (device globals start zeroed).  A load that falls
// outside the matrix or past the part end reads this instead, so that no
// instruction touches a loaded value before it is stored -- a select on the
// loaded value would make the load wait at once.
static __device__ u32x4 g_zero16[1];

__device__ __forceinline__ const u32x4* chunk_or_zero(bool ok, const uint16_t* p) {
  return ok ? reinterpret_cast<const u32x4*>(p) : &g_zero16[0];
}

// Odd-sized operands (UN, "unaligned": K, N, the part starts and the pointers
// any multiple of an element).  A chunk is still 8 consecutive elements and
// one 16-byte load, at whatever address it has; rows are not padded, so a
// chunk that crosses its row's end holds the next row's first elements, in
// bounds.  Columns past N only feed outputs that are not stored.  In a part's
// last slab, before the chunks go to LDS, elements of A at or past the part
// end are cleared (B's rows there are zero chunks, and 0 x NaN must not
// arise), and the one chunk of each matrix whose 16 bytes would run past its
// end (which is never loaded) is put together from single elements.  With
// N, K >= 8 that chunk is in the last row, so in the last slab.
typedef u32x4 u32x4u __attribute__((aligned(2)));
typedef floatx4 floatx4u __attribute__((aligned(4)));
typedef u32x2 u32x2u __attribute__((aligned(2)));

template <bool UN>
__device__ __forceinline__ u32x4 load_chunk(bool ok, const uint16_t* p) {
  if constexpr (UN) return *(ok ? reinterpret_cast<const u32x4u*>(p) : reinterpret_cast<const u32x4u*>(&g_zero16[0]));
  else return *chunk_or_zero(ok, p);
}

// The first n of a chunk's 8 elements, zeros after them.
__device__ __forceinline__ u32x4 keep_elems(u32x4 v, int n) {
#pragma unroll
  for (int w = 0; w < 4; ++w) v[w] = n >= 2 * w + 2 ? v[w] : n == 2 * w + 1 ? (v[w] & 0xffffu) : 0u;
  return v;
}

// n (1 to 8) elements from p, one by one, zeros after them.
__device__ __forceinline__ u32x4 load_elems(const uint16_t* p, int n) {
  u32x4 v;
#pragma unroll
  for (int w = 0; w < 4; ++w)
    v[w] = (2 * w < n ? (uint32_t)p[2 * w] : 0u) | (2 * w + 1 < n ? (uint32_t)p[2 * w + 1] << 16 : 0u);
  return v;
}

// A chunk of the part's last slab as it goes to LDS: A at (gi, gk), B at (gk, gn).
__device__ __forceinline__ u32x4 last_a(const GemmArgs& a, u32x4 v, int64_t gi, int64_t gk, int64_t k1) {
  if (gi < a.M && gk < k1) {
    const int n = k1 - gk < 8 ? (int)(k1 - gk) : 8;
    if (gi * a.K + gk + 8 > a.M * a.K) v = load_elems(a.A + gi * a.K + gk, n);
    else v = keep_elems(v, n);
  }
  return v;
}
__device__ __forceinline__ u32x4 last_b(const GemmArgs& a, u32x4 v, int64_t gk, int64_t gn, int64_t k1) {
  if (gk < k1 && gn < a.N && gk * a.N + gn + 8 > a.K * a.N) v = load_elems(a.B + gk * a.N + gn, (int)(a.N - gn));
  return v;
}
// Whether a chunk may be loaded whole (UN; else every chunk is inside or outside).
template <bool UN>
__device__ __forceinline__ bool whole_a(const GemmArgs& a, int64_t gi, int64_t gk) {
  return !UN || gi * a.K + gk + 8 <= a.M * a.K;
}
template <bool UN>
__device__ __forceinline__ bool whole_b(const GemmArgs& a, int64_t gk, int64_t gn) {
  return !UN || gk * a.N + gn + 8 <= a.K * a.N;
}

// LDS layout of A slabs ([row][k], CPR 16-byte chunks per row): chunk c of
// row r sits at position c ^ swz_a<CPR>(r).  A fragment read takes one chunk
// of 16 consecutive rows; with 64-byte rows (CPR 4) the swizzle gives every
// 8 consecutive rows distinct 16-byte slots of a 128-byte bank window and
// every 16 rows distinct slots of a 256-byte one (with 128-byte rows, CPR 8,
// likewise one row per 128 bytes), so the read has no bank conflict whether
// the LDS serves 8 or 16 lanes per pass.  Measured on the MLP kernel: bank
// conflict cycles fell from 1.7e7 to 4.6e5 and the kernel's cycles by 9 %
// against the earlier swizzle c ^ ((r / 4) mod 4).
template <int CPR>
__device__ __forceinline__ int swz_a(int row) {
  static_assert(CPR == 4 || CPR == 8, "64- or 128-byte rows");
  constexpr int sh = CPR == 4 ? 1 : 0;
  return ((row >> sh) ^ (row >> (sh + 1))) & (CPR - 1);
}



// finish() for four consecutive columns j..j+3 (all < N: the tiled path
// requires N % 8 == 0 and 16-byte aligned C), with one vector store; b4 holds
// the bias of those columns as binary32 (used only by the epilogue).  Returns
// the four values as stored in C, as binary32 (the partials when S > 1).
// UN: N and C any; columns at or past N are not stored.
template <bool UN = false>
__device__ __forceinline__ float4 finish4v(const GemmArgs& a, int s, int64_t i, int64_t j, float4 y4, float4 b4) {
  float y[4] = {y4.x, y4.y, y4.z, y4.w};
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (a.partial_bf16) y[e] = round_bf16(y[e]);
  const int nc = UN && a.N - j < 4 ? (int)(a.N - j) : 4;
  auto put_f32 = [&](float* p) {
    if constexpr (!UN) {
      *(float4*)p = float4{y[0], y[1], y[2], y[3]};
    } else if (nc == 4) {
      *(floatx4u*)p = floatx4{y[0], y[1], y[2], y[3]};
    } else {
      p[0] = y[0];
      if (nc > 1) p[1] = y[1];
      if (nc > 2) p[2] = y[2];
    }
  };
  if (a.S > 1) {
    put_f32(&a.ws[((int64_t)s * a.M + i) * a.N + j]);
    return float4{y[0], y[1], y[2], y[3]};
  }
  if (a.epilogue != DG_EPI_NONE) {
    const float b[4] = {b4.x, b4.y, b4.z, b4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = y[e] + b[e];
  }
  if (a.epilogue == DG_EPI_BIAS_SILU) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float z = y[e];
      if (a.pre_act) z = round_bf16(z);
      y[e] = silu_f32(z);
    }
  }
  if (a.out_bf16) {
    const uint32_t lo = f32x2_bf16x2(y[0], y[1]);
    const uint32_t hi = f32x2_bf16x2(y[2], y[3]);
    uint16_t* p = &((uint16_t*)a.C)[i * a.N + j];
    if constexpr (!UN) {
      *(uint2*)p = uint2{lo, hi};
    } else if (nc == 4) {
      *(u32x2u*)p = u32x2{lo, hi};
    } else {
      p[0] = (uint16_t)lo;
      if (nc > 1) p[1] = (uint16_t)(lo >> 16);
      if (nc > 2) p[2] = (uint16_t)hi;
    }
    return float4{bits_f32(lo << 16), bits_f32(lo & 0xffff0000u), bits_f32(hi << 16), bits_f32(hi & 0xffff0000u)};
  }
  put_f32(&((float*)a.C)[i * a.N + j]);
  return float4{y[0], y[1], y[2], y[3]};
}

// finish4v with the bias read from memory.
template <bool UN = false>
__device__ __forceinline__ void finish4(const GemmArgs& a, int s, int64_t i, int64_t j, float4 y4) {
  float4 b4 = float4{0.f, 0.f, 0.f, 0.f};
  if (UN && a.S == 1 && a.epilogue != DG_EPI_NONE) {
    b4.x = bf16_f32(a.bias[j]);
    if (j + 1 < a.N) b4.y = bf16_f32(a.bias[j + 1]);
    if (j + 2 < a.N) b4.z = bf16_f32(a.bias[j + 2]);
    if (j + 3 < a.N) b4.w = bf16_f32(a.bias[j + 3]);
  } else if (a.S == 1 && a.epilogue != DG_EPI_NONE) {
    const uint2 bb = *(const uint2*)&a.bias[j];
    b4 = float4{bits_f32(bb.x << 16), bits_f32(bb.x & 0xffff0000u), bits_f32(bb.y << 16), bits_f32(bb.y & 0xffff0000u)};
  }
  (void)finish4v<UN>(a, s, i, j, y4, b4);
}

// Whether the epilogue reads the bias (a single part, bias epilogue).
__device__ __forceinline__ bool needs_bias(const GemmArgs& a) { return a.S == 1 && a.epilogue != DG_EPI_NONE; }

// The bias of columns [j0, j0 + n) as binary32 into LDS (zero past N), by
// all threads of the workgroup; the caller synchronises afterwards.
__device__ __forceinline__ void stage_bias(const GemmArgs& a, int64_t j0, int n, float* bsh) {
  if (!needs_bias(a)) return;
  for (int c = threadIdx.x; c < n; c += blockDim.x) bsh[c] = j0 + c < a.N ? bf16_f32(a.bias[j0 + c]) : 0.f;
}

// Wait for the wave's own LDS operations (and keep the compiler from moving
// memory operations across).  LDS operations of one wave run in issue order,
// so after this a read sees what the wave wrote before.
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Epilogue of one wave's (16 TM) x (16 TN) tile of 16x16 MFMA accumulators
// (lane l holds rows 4 (l / 16) .. +3, column l % 16 of each), rows from ib
// and columns from jb.  Each 16-row band passes through the wave's own LDS
// area cs (16 rows of pitch 16 TN + 4 floats: rows 4 apart start 16 banks
// apart) and leaves as four-column vectors; the bias of the wave's columns
// comes from bsh (staged by stage_bias), so no global load waits inside the
// loop.  Only the wave itself touches cs, so no workgroup barrier is needed.
// With croot set, the wave also folds each of its columns down its 16 TM
// rows as the perfect tree of the values stored in C (rows past M count as
// -0, the exact identity): the band's values go back into cs, lane c takes
// column c of the band (rows paired from the top, 16-row band roots paired
// the same way), and the root lands in croot[c].
template <int TM, int TN, bool UN = false, typename Acc>
__device__ __forceinline__ void wave_epilogue(const GemmArgs& a, int s, int64_t ib, int64_t jb, float* cs,
                                              const float* bsh, const Acc& acc, float* croot = nullptr) {
  constexpr int WTN = 16 * TN, CSP = WTN + 4;
  static_assert((TM & (TM - 1)) == 0, "a power-of-two band count");
  const int lane = threadIdx.x & 63;
  const bool bias = needs_bias(a), tree = WTN <= 64 && croot != nullptr;   // one column per lane
  float band[TM];
#pragma unroll
  for (int mi = 0; mi < TM; ++mi) {
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
      for (int r = 0; r < 4; ++r) cs[(4 * (lane >> 4) + r) * CSP + 16 * ni + (lane & 15)] = acc[mi][ni][r];
    lds_wait();
#pragma unroll 1
    for (int q = lane; q < 16 * WTN / 4; q += 64) {
      const int rr = q / (WTN / 4), cc = 4 * (q % (WTN / 4));
      const int64_t i = ib + 16 * mi + rr, j = jb + cc;
      float4* p = (float4*)&cs[rr * CSP + cc];
      const float4 y4 = *p;
      const float4 b4 = bias ? *(const float4*)&bsh[cc] : float4{0.f, 0.f, 0.f, 0.f};
      float4 v = float4{-0.f, -0.f, -0.f, -0.f};
      if (i < a.M && j < a.N) v = finish4v<UN>(a, s, i, j, y4, b4);
      if (tree) *p = v;
    }
    lds_wait();
    if (WTN <= 64 && tree) {
      float v[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) v[r] = lane < WTN ? cs[r * CSP + lane] : 0.f;
#pragma unroll
      for (int w = 1; w < 16; w <<= 1)
#pragma unroll
        for (int r = 0; r < 16; r += 2 * w) v[r] = v[r] + v[r + w];
      band[mi] = v[0];
      lds_wait();
    }
  }
  if (WTN <= 64 && tree) {
#pragma unroll
    for (int w = 1; w < TM; w <<= 1)
#pragma unroll
      for (int mi = 0; mi < TM; mi += 2 * w) band[mi] = band[mi] + band[mi + w];
    if (lane < WTN) croot[lane] = band[0];
  }
}

// ------------------------------------------------------------ tiled v3
//
// Same order as gemm_tiled (16x16x32 MFMA chain, 8-k chunks from k = 0), with
// a deeper, branch-free pipeline:
//   * A and B live in LDS in their global row-major layouts ([m][k], [k][n]),
//     16-byte chunks XOR-swizzled per row so that fragment reads spread over
//     the banks; B fragments come out of LDS already transposed through
//     ds_read_b64_tr_b16 (a 16-lane group reading rows k0..k0+3, 4 columns
//     per lane, hands lane j column j of those 4 rows);
//   * every chunk is either wholly inside the part and the matrix or wholly
//     outside (part ends and N are multiples of 8), so a load is a select
//     between a 16-byte load and zero, with no branches;
//   * global loads run two 64-k slabs ahead through a ring of two register
//     sets, into an LDS double buffer, one barrier per slab.
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) shortx4* lds_s4;

// The same pipeline serves the descriptors whose accumulator is not one
// carried chain (tile_combine chain or tree, or fma = 0) when every tile
// boundary lies on a 32-k step from the part start: COMB is the tile
// combine, FMA0 that each 32-k instruction starts from zero and its result
// is added to the tile's accumulator (v = v + w, one binary32 addition per
// element), L the levels of the tile tree's binary-counter stack, held in
// registers.  The part's last tile stays in the accumulator (its folded
// value is the lowest entry of the final fold) and needs no level of its
// own, so L levels hold a part of up to 2^L tiles.  Steps past the part end are skipped, so they close no tile and
// add nothing.
template <int BM, int BN, int WM, int WN, int V3_BK, bool F16, int COMB = DG_CARRY, bool FMA0 = false, int L = 1,
          bool UN = false>
__device__ __forceinline__ void v3_body(const GemmArgs& a, int64_t i0, int64_t j0) {
  static_assert(WM * WN == 4, "four waves");
  constexpr bool GEN = COMB != DG_CARRY || FMA0;   // not one carried chain
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 16, TN = WTN / 16;
  constexpr int ACH = BM * (V3_BK / 8);        // 16-byte chunks per A slab
  constexpr int BCH = V3_BK * (BN / 8);        // 16-byte chunks per B slab
  constexpr int ACH_T = ACH / 256, BCH_T = BCH / 256;
  static_assert(ACH % 256 == 0 && BCH % 256 == 0, "whole chunks per thread");
  constexpr int A_ELEMS = BM * V3_BK, B_ELEMS = V3_BK * BN;   // bf16 per stage
  constexpr int BROW = BN / 8;                 // chunks per B row

  __shared__ __attribute__((aligned(16))) uint16_t smem[2 * (A_ELEMS + B_ELEMS)];
  uint16_t* As0 = smem;
  uint16_t* Bs0 = smem + 2 * A_ELEMS;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int s = blockIdx.z;
  const int64_t k0 = a.cuts[s], k1 = a.cuts[s + 1];
  const int nslab = (int)((k1 - k0 + V3_BK - 1) / V3_BK);

  // A chunk (row, c): LDS chunk row*CPR + (c ^ swz_a<CPR>(row)), CPR = chunks per
  // row (conflict-free fragment reads, as the swizzle's own comment says).
  // B chunk (k, c): LDS chunk k*BROW + (c ^ ((k & 3) << 1)) -- the four rows a
  // transpose read touches land on four different 32-byte bank groups.
  constexpr int CPR = V3_BK / 8;
  static_assert(CPR == 4 || CPR == 8, "BK 32 or 64");
  auto ldsA = [](int row, int c) { return row * CPR + (c ^ swz_a<CPR>(row)); };
  auto ldsB = [](int k, int c) { return k * BROW + (c ^ ((k & 3) << 1)); };

  u32x4 r0a[ACH_T], r0b[BCH_T], r1a[ACH_T], r1b[BCH_T];
  auto gload = [&](int sl, u32x4* ra, u32x4* rb) {
    const int64_t ks = k0 + (int64_t)sl * V3_BK;
#pragma unroll
    for (int t = 0; t < ACH_T; ++t) {
      const int q = tid + 256 * t, row = q / (V3_BK / 8), c = q % (V3_BK / 8);
      const int64_t gi = i0 + row, gk = ks + 8 * c;
      ra[t] = load_chunk<UN>((gi < a.M) && (gk < k1) && whole_a<UN>(a, gi, gk), a.A + gi * a.K + gk);
    }
#pragma unroll
    for (int t = 0; t < BCH_T; ++t) {
      const int q = tid + 256 * t, kr = q / BROW, c = q % BROW;
      const int64_t gk = ks + kr, gn = j0 + 8 * c;
      rb[t] = load_chunk<UN>((gk < k1) && (gn < a.N) && whole_b<UN>(a, gk, gn), a.B + gk * a.N + gn);
    }
  };
  auto lstore = [&](int buf, int sl, u32x4* ra, u32x4* rb) {
    uint16_t* As = As0 + buf * A_ELEMS;
    uint16_t* Bs = Bs0 + buf * B_ELEMS;
    if (UN && sl == nslab - 1) {
      const int64_t ks = k0 + (int64_t)sl * V3_BK;
#pragma unroll
      for (int t = 0; t < ACH_T; ++t) {
        const int q = tid + 256 * t;
        ra[t] = last_a(a, ra[t], i0 + q / (V3_BK / 8), ks + 8 * (q % (V3_BK / 8)), k1);
      }
#pragma unroll
      for (int t = 0; t < BCH_T; ++t) {
        const int q = tid + 256 * t;
        rb[t] = last_b(a, rb[t], ks + q / BROW, j0 + 8 * (q % BROW), k1);
      }
    }
#pragma unroll
    for (int t = 0; t < ACH_T; ++t) {
      const int q = tid + 256 * t;
      *(u32x4*)&As[8 * ldsA(q / (V3_BK / 8), q % (V3_BK / 8))] = ra[t];
    }
#pragma unroll
    for (int t = 0; t < BCH_T; ++t) {
      const int q = tid + 256 * t;
      *(u32x4*)&Bs[8 * ldsB(q / BROW, q % BROW)] = rb[t];
    }
  };

  floatx4 acc[TM][TN];
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = floatx4{0.f, 0.f, 0.f, 0.f};

  // tile combine state (GEN only): the open tile's accumulator is acc; the
  // chain's running sum or the tree's stack hold the closed tiles
  constexpr int NL = COMB == DG_TREE ? L : COMB == DG_SEQ ? 1 : 0;
  floatx4 stk[NL > 0 ? NL : 1][TM][TN];
  uint32_t count = 0;                                  // tiles closed
  int64_t tile_end = k1;                               // end of the open tile
  if constexpr (GEN) {
    const int64_t len = k1 - k0, tk = a.tile_k;
    const int64_t first = (a.tail_first && len % tk) ? len % tk : tk;
    tile_end = k0 + (first < len ? first : len);
  }
  const floatx4 zero4 = {0.f, 0.f, 0.f, 0.f};
  auto close_tile = [&](bool last) {
    if constexpr (COMB == DG_SEQ) {
      if (count == 0) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
          for (int ni = 0; ni < TN; ++ni) stk[0][mi][ni] = acc[mi][ni];
      } else {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
          for (int ni = 0; ni < TN; ++ni) stk[0][mi][ni] = stk[0][mi][ni] + acc[mi][ni];
      }
    } else if constexpr (COMB == DG_TREE) {
      // binary counter: fold the levels whose bit is set, park at the first clear one
      bool parked = false;
      static_for<0, NL>([&](auto lv) {
        constexpr int LV = decltype(lv)::value;
        if (!parked) {
          if ((count >> LV) & 1u) {
#pragma unroll
            for (int mi = 0; mi < TM; ++mi)
#pragma unroll
              for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = stk[LV][mi][ni] + acc[mi][ni];
          } else {
#pragma unroll
            for (int mi = 0; mi < TM; ++mi)
#pragma unroll
              for (int ni = 0; ni < TN; ++ni) stk[LV][mi][ni] = acc[mi][ni];
            parked = true;
          }
        }
      });
    }
    ++count;
    if (COMB == DG_SEQ || !last) {
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = zero4;
    }
  };

  auto compute = [&](int buf, int sl) {
    const uint16_t* As = As0 + buf * A_ELEMS;
    const uint16_t* Bs = Bs0 + buf * B_ELEMS;
#pragma unroll
    for (int kk = 0; kk < V3_BK; kk += 32) {
      shortx8 af[TM], bfr[TN];
#pragma unroll
      for (int mi = 0; mi < TM; ++mi) {
        const int row = wm * WTM + 16 * mi + (lane & 15);
        af[mi] = *(const shortx8*)&As[8 * ldsA(row, kk / 8 + (lane >> 4))];
      }
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        const int i = lane & 15, g = lane >> 4;
        const int n = wn * WTN + 16 * ni + 4 * (i & 3);
        const int kr0 = kk + 8 * g + (i >> 2), kr1 = kr0 + 4;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s4)(&Bs[8 * ldsB(kr0, n / 8) + (n & 7)]));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_s4)(&Bs[8 * ldsB(kr1, n / 8) + (n & 7)]));
        bfr[ni] = shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      }
      if constexpr (!GEN) {
#pragma unroll
        for (int mi = 0; mi < TM; ++mi)
#pragma unroll
          for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = mfma16t<F16>(af[mi], bfr[ni], acc[mi][ni]);
      } else {
        const int64_t kpos = k0 + (int64_t)sl * V3_BK + kk;   // this 32-k step (uniform)
        if (kpos < k1) {
#pragma unroll
          for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) {
              if constexpr (FMA0) {
                const floatx4 w = mfma16t<F16>(af[mi], bfr[ni], zero4);
                acc[mi][ni] = acc[mi][ni] + w;
              } else {
                acc[mi][ni] = mfma16t<F16>(af[mi], bfr[ni], acc[mi][ni]);
              }
            }
          if constexpr (COMB != DG_CARRY) {
            if (kpos + 32 >= tile_end) {
              close_tile(tile_end >= k1);
              tile_end = tile_end + a.tile_k < k1 ? tile_end + a.tile_k : k1;
            }
          }
        }
      }
    }
  };

  // prologue: slabs 0 and 1 in flight, slab 0 in LDS.  Loads and LDS
  // stores are unconditional (past the part end they read the zero chunk) so
  // that the store of a slab waits only for that slab's loads.
  gload(0, r0a, r0b);
  gload(1, r1a, r1b);
  lstore(0, 0, r0a, r0b);
  __syncthreads();
  for (int sl = 0; sl < nslab; sl += 2) {
    // even slab sl in buffer 0, its successor's registers in set 1
    gload(sl + 2, r0a, r0b);
    compute(0, sl);
    lstore(1, sl + 1, r1a, r1b);
    __syncthreads();
    gload(sl + 3, r1a, r1b);
    if (sl + 1 < nslab) compute(1, sl + 1);
    lstore(0, sl + 2, r0a, r0b);
    __syncthreads();
  }
  // the part's value: the chain's sum, or the tree's stack folded low to high
  if constexpr (COMB == DG_SEQ) {
    if (count) {
#pragma unroll
      for (int mi = 0; mi < TM; ++mi)
#pragma unroll
        for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = stk[0][mi][ni];
    }
  } else if constexpr (COMB == DG_TREE) {
    // acc holds the last tile's folded value, the entry of level ctz(count);
    // the set levels above it meet it in increasing order
    if (count) {
      const int low = __builtin_ctz(count);
      static_for<0, NL>([&](auto lv) {
        constexpr int LV = decltype(lv)::value;
        if (LV > low && ((count >> LV) & 1u)) {
#pragma unroll
          for (int mi = 0; mi < TM; ++mi)
#pragma unroll
            for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = stk[LV][mi][ni] + acc[mi][ni];
        }
      });
    }
  }

  // staging rows of pitch WTN + 4 floats: the four row groups a write
  // instruction covers (rows 4 apart) start 16 banks apart
  constexpr int CSP = WTN + 4;
  float* cs = reinterpret_cast<float*>(smem) + wave * 16 * CSP;
  static_assert(4 * 16 * CSP * 4 <= (int)sizeof(smem), "epilogue staging fits");
#pragma unroll
  for (int mi = 0; mi < TM; ++mi) {
    __syncthreads();
#pragma unroll
    for (int ni = 0; ni < TN; ++ni)
#pragma unroll
      for (int r = 0; r < 4; ++r) cs[(4 * (lane >> 4) + r) * CSP + 16 * ni + (lane & 15)] = acc[mi][ni][r];
    __syncthreads();
#pragma unroll 1
    for (int q = lane; q < 16 * WTN / 4; q += 64) {
      const int rr = q / (WTN / 4), cc = 4 * (q % (WTN / 4));
      const int64_t i = i0 + wm * WTM + 16 * mi + rr, j = j0 + wn * WTN + cc;
      if (i < a.M && j < a.N) finish4<UN>(a, s, i, j, *(const float4*)&cs[rr * CSP + cc]);
    }
  }
}

// Block order (speed only).  order 1: row-major, consecutive workgroups share
// an A panel.  order 2: groups of eight block rows walked column by column.
// order 3: as 2, after giving each XCD (workgroup w runs on XCD w % 8) a
// contiguous range of blocks, so that one XCD's L2 sees neighbouring panels.
__device__ __forceinline__ void grouped_tile(int w, int tiles_m, int tiles_n, int order, int* ty, int* tx) {
  if (order <= 1) {
    *ty = w / tiles_n;
    *tx = w % tiles_n;
    return;
  }
  const int nwg = tiles_m * tiles_n;
  if (order == 3 && nwg % 8 == 0) w = (w % 8) * (nwg / 8) + w / 8;
  constexpr int GROUP = 8;
  const int group = w / (GROUP * tiles_n);
  const int first = group * GROUP;
  const int rows = (tiles_m - first < GROUP) ? tiles_m - first : GROUP;
  const int in_group = w - group * GROUP * tiles_n;
  *ty = first + in_group % rows;
  *tx = in_group / rows;
}

// ------------------------------------------------- ping-pong (eight waves)
//
// Two groups of four waves (one wave of each group per SIMD).  Group g owns
// rows [g BM/2, (g+1) BM/2) of the BM x BN block; each wave a (BM/2) x (BN/4)
// sub-tile.  The groups run the same sequence of phases one phase apart, a
// barrier closing every phase, so that on each SIMD one wave issues MFMAs
// while the other works on LDS:
//   memory phase of slab s: write the group's half of slab s+1 to LDS from
//     registers, read the wave's fragments of slab s;
//   compute phase of slab s: the MFMAs of slab s (its 32-k halves in order),
//     with the loads of the group's half of slab s+3 spread among them (into
//     the register set just written to LDS; two sets alternate).
// Slab s+1's halves are written in phases 2s and 2s+1 and first read in
// phase 2s+2; its buffer last held slab s-1, last read in phase 2s-1.  The
// group that starts late and the group that ends early each take one barrier
// on their own, so every wave takes the same number of barriers.  Slabs past
// the part end are all zero chunks, whose MFMAs leave the accumulators' bits
// unchanged.
//
// Global loads go through buffer resources: a thread's byte offsets inside
// the block are fixed for the launch (a row past M or a column past N gets
// an offset past the resource's end, which reads zero), the slab moves a
// scalar offset, and chunks are checked against the part end only through a
// compare with the elements left.  The host guarantees every offset fits 31
// bits.
// BNC <= BN is the number of columns the block computes; the B slab keeps
// the BN-wide LDS layout and load mapping, and its chunks past BNC are
// neither loaded nor stored.
template <int BM, int BN, int BK, int BNC, bool F16, bool UN = false>
__device__ __forceinline__ void pp_body(const GemmArgs& a, int64_t i0, int64_t j0, uint16_t* smem) {
  constexpr int CPR = BK / 8, KK = BK / 32, WTM = BM / 2, WTN = BNC / 4, TM = WTM / 16, TN = WTN / 16;
  constexpr int BROW = BN / 8;
  constexpr int ACH_T = (BM / 2) * CPR / 256, BCH_T = (BK / 2) * BROW / 256;   // per thread
  constexpr int NLOAD = ACH_T + BCH_T, NPAIR = KK * TM;
  static_assert((BM / 2) * CPR % 256 == 0 && (BK / 2) * BROW % 256 == 0 && BROW >= 16, "whole chunks");
  static_assert(CPR == 4 || CPR == 8, "32- or 64-k slabs");
  static_assert(NPAIR >= NLOAD, "at most one load per MFMA group");
  static_assert(BNC <= BN && BNC % 64 == 0, "whole 16-column fragments per wave");
  constexpr int A_ELEMS = BM * BK, B_ELEMS = BK * BN;
  uint16_t* As0 = smem;
  uint16_t* Bs0 = smem + 2 * A_ELEMS;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int grp = wave >> 2, wn = wave & 3, tg = tid & 255;
  const int s = blockIdx.z;
  const int64_t k0 = a.cuts[s], k1 = a.cuts[s + 1];
  const int nslab = (int)((k1 - k0 + BK - 1) / BK);
  // A: chunk c of row r at c ^ swz_a<CPR>(r); B: chunk c of
  // k-row k at c ^ 2 (k % 4) ^ 8 ((k / 8) % 2)
  auto ldsA = [](int row, int c) { return row * CPR + (c ^ swz_a<CPR>(row)); };
  auto ldsB = [](int k, int c) { return k * BROW + (c ^ ((k & 3) << 1) ^ (((k >> 3) & 1) << 3)); };

  constexpr uint32_t OOB = 0x80000000u;
  // UN: the resources start on 16 bytes, mis* bytes before the operands' own start
  const uint16_t *pA = a.A + i0 * a.K, *pB = a.B + k0 * a.N;
  const uint32_t misA = UN ? (uint32_t)((uintptr_t)pA & 15) : 0, misB = UN ? (uint32_t)((uintptr_t)pB & 15) : 0;
  const int64_t recA = (a.M - i0) * a.K * 2 + misA, recB = (a.K - k0) * a.N * 2 + misB;
  const __amdgpu_buffer_rsrc_t rA = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const char*)pA - misA), (short)0, (int)(recA < 0x7fffffff ? recA : 0x7fffffff), 0x00020000);
  const __amdgpu_buffer_rsrc_t rB = __builtin_amdgcn_make_buffer_rsrc(
      (void*)((const char*)pB - misB), (short)0, (int)(recB < 0x7fffffff ? recB : 0x7fffffff), 0x00020000);
  // the group's half of a slab: A rows [grp BM/2, +BM/2), B k-rows [grp BK/2, +BK/2)
  uint32_t offA[ACH_T], offB[BCH_T];
  int kcA[ACH_T], kcB[BCH_T];   // the chunk's k within the slab
  int ldA[ACH_T], ldB[BCH_T];   // its LDS chunk
#pragma unroll
  for (int t = 0; t < ACH_T; ++t) {
    const int q = tg + 256 * t, row = grp * (BM / 2) + q / CPR, c = q % CPR;
    offA[t] = (i0 + row < a.M) ? (uint32_t)((row * a.K + 8 * c) * 2) + misA : OOB;
    kcA[t] = 8 * c;
    ldA[t] = ldsA(row, c);
  }
#pragma unroll
  for (int t = 0; t < BCH_T; ++t) {
    const int q = tg + 256 * t, kr = grp * (BK / 2) + q / BROW, c = q % BROW;
    offB[t] = (8 * c < BNC && j0 + 8 * c < a.N) ? (uint32_t)((kr * a.N + j0 + 8 * c) * 2) + misB : OOB;
    kcB[t] = kr;
    ldB[t] = 8 * c < BNC ? ldsB(kr, c) : -1;
  }
  u32x4 ga2[2][ACH_T], gb2[2][BCH_T];
  // load number t of the thread's share of slab sl (A chunks first)
  auto gload1 = [&](int sl, int t, u32x4* ga, u32x4* gb) {
    const int64_t ks = k0 + (int64_t)sl * BK, lim = k1 - ks;
    if (t < ACH_T) {
      const uint32_t off = kcA[t] < lim ? offA[t] : OOB;
      ga[t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rA, off, (int)(ks * 2), 0));
    } else {
      const int u = t - ACH_T;
      const uint32_t off = kcB[u] < lim ? offB[u] : OOB;
      gb[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rB, off, (int)((ks - k0) * a.N * 2), 0));
    }
  };
  auto gload = [&](int sl, u32x4* ga, u32x4* gb) {
#pragma unroll
    for (int t = 0; t < NLOAD; ++t) gload1(sl, t, ga, gb);
  };
  auto lstore = [&](int buf, int sl, u32x4* ga, u32x4* gb) {
    uint16_t* As = As0 + buf * A_ELEMS;
    uint16_t* Bs = Bs0 + buf * B_ELEMS;
    if (UN && sl == nslab - 1) {
      const int64_t ks = k0 + (int64_t)sl * BK;
#pragma unroll
      for (int t = 0; t < ACH_T; ++t)
        ga[t] = last_a(a, ga[t], i0 + grp * (BM / 2) + (tg + 256 * t) / CPR, ks + kcA[t], k1);
#pragma unroll
      for (int t = 0; t < BCH_T; ++t) {
        const int c = (tg + 256 * t) % BROW;
        if (8 * c < BNC) gb[t] = last_b(a, gb[t], ks + kcB[t], j0 + 8 * c, k1);
      }
    }
#pragma unroll
    for (int t = 0; t < ACH_T; ++t) *(u32x4*)&As[8 * ldA[t]] = ga[t];
#pragma unroll
    for (int t = 0; t < BCH_T; ++t)
      if (BNC == BN || ldB[t] >= 0) *(u32x4*)&Bs[8 * ldB[t]] = gb[t];
  };

  floatx4 acc[TM][TN];
#pragma unroll
  for (int mi = 0; mi < TM; ++mi)
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = floatx4{0.f, 0.f, 0.f, 0.f};

  shortx8 af[KK][TM], bf[KK][TN];
  auto rd = [&](int buf) {
    const uint16_t* As = As0 + buf * A_ELEMS;
    const uint16_t* Bs = Bs0 + buf * B_ELEMS;
#pragma unroll
    for (int h = 0; h < KK; ++h) {
#pragma unroll
      for (int ni = 0; ni < TN; ++ni) {
        const int i = lane & 15, g = lane >> 4;
        const int n = wn * WTN + 16 * ni + 4 * (i & 3);
        const int kr0 = 32 * h + 8 * g + (i >> 2), kr1 = kr0 + 4;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&Bs[8 * ldsB(kr0, n / 8) + (n & 7)]));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&Bs[8 * ldsB(kr1, n / 8) + (n & 7)]));
        bf[h][ni] = shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      }
#pragma unroll
      for (int mi = 0; mi < TM; ++mi) {
        const int row = grp * WTM + 16 * mi + (lane & 15);
        af[h][mi] = *(const shortx8*)&As[8 * ldsA(row, 4 * h + (lane >> 4))];
      }
    }
  };
  // MFMAs of pair p: 32-k half p / TM, fragment row p % TM (halves in order)
  auto mm_pair = [&](int p) {
    const int h = p / TM, mi = p % TM;
#pragma unroll
    for (int ni = 0; ni < TN; ++ni) acc[mi][ni] = mfma16t<F16>(af[h][mi], bf[h][ni], acc[mi][ni]);
  };

  // prologue: slab 0 in buffer 0, slabs 1 and 2 in the two register sets
  gload(0, ga2[0], gb2[0]);
  lstore(0, 0, ga2[0], gb2[0]);
  gload(1, ga2[1], gb2[1]);
  gload(2, ga2[0], gb2[0]);
  __syncthreads();
  if (grp == 1) __syncthreads();
  auto step = [&](int sl, u32x4* ga, u32x4* gb) {
    // memory phase: ga/gb hold slab sl+1
    __builtin_amdgcn_sched_barrier(0);
    lstore((sl + 1) & 1, sl + 1, ga, gb);
    rd(sl & 1);
    __syncthreads();
    // compute phase; ga/gb are refilled with slab sl+3
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(2);
    // load l goes after MFMA group (l + 1) NPAIR / NLOAD - 1
    static_for<0, NPAIR>([&](auto p) {
      mm_pair(p);
      static_for<0, NLOAD>([&](auto l) {
        if constexpr ((l + 1) * NPAIR / NLOAD - 1 == p) {
          __builtin_amdgcn_sched_barrier(0);
          gload1(sl + 3, l, ga, gb);
          __builtin_amdgcn_sched_barrier(0);
        }
      });
    });
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
  };
  for (int sl = 0; sl < nslab; sl += 2) {
    step(sl, ga2[1], gb2[1]);
    step(sl + 1, ga2[0], gb2[0]);
  }
  if (grp == 0) __syncthreads();

  constexpr int CSP = WTN + 4;
  float* cs = reinterpret_cast<float*>(smem) + wave * 16 * CSP;
  float* bsh = reinterpret_cast<float*>(smem) + 8 * 16 * CSP;
  float* croot = bsh + BNC;   // [group][column]: each group's column roots
  static_assert((8 * 16 * CSP + 3 * BNC) * 4 <= 2 * (A_ELEMS + B_ELEMS) * 2, "epilogue staging fits");
  __syncthreads();
  stage_bias(a, j0, BNC, bsh);
  __syncthreads();
  // a 256-row block is one run of the column sums: each group folds its 128
  // rows, and the two roots meet (group 0's rows first)
  const bool tree = BM == 256 && a.colsum_part != nullptr;
  wave_epilogue<TM, TN, UN>(a, s, i0 + grp * WTM, j0 + wn * WTN, cs, bsh + wn * WTN, acc,
                        tree ? croot + grp * BNC + wn * WTN : nullptr);
  if (tree) {
    __syncthreads();
    for (int c = tid; c < BNC; c += 512)
      if (j0 + c < a.N) a.colsum_part[(i0 / 256) * a.N + j0 + c] = croot[c] + croot[BNC + c];
  }
}

// ---------------------------------------------------------- skinny (M <= 64)
//
// Few rows: the GEMM streams B from HBM and the MFMA work per slab is small,
// so the time goes to memory latency.  Each workgroup owns BN columns (one
// 16-column MFMA tile per computing wave, all four waves loading) and keeps
// D BK-k slabs of loads in flight through a ring of D register sets, staged
// through an LDS double buffer in the layouts of the v3 kernel (A [m][k], B
// [k][n], transposing reads for B).  Same chunk order as every other path.
// When the column tiles split evenly over the eight XCDs (workgroup w runs
// on XCD w mod 8), each XCD takes a contiguous range of them, so that tiles
// sharing 128-byte B lines share an L2.
template <int TMS, int BN, int D, int BK, bool F16, bool UN = false>
__device__ __forceinline__ void skinny_body(const GemmArgs& a) {
  constexpr int CPR = BK / 8, BM = 16 * TMS, NWC = BN / 16;
  constexpr int ACH = BM * CPR, BCH = BK * (BN / 8), BROW = BN / 8;
  constexpr int ACH_T = (ACH + 255) / 256, BCH_T = (BCH + 255) / 256;
  constexpr int A_ELEMS = BM * BK, B_ELEMS = BK * BN;
  static_assert(BN % 64 == 0 || BN == 16 || BN == 32, "B rows of whole swizzle blocks");
  __shared__ __attribute__((aligned(16))) uint16_t smem[2 * (A_ELEMS + B_ELEMS)];
  uint16_t* As0 = smem;
  uint16_t* Bs0 = smem + 2 * A_ELEMS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nt = gridDim.x, x = blockIdx.x;
  const int tile = (nt % 8 == 0) ? (x % 8) * (nt / 8) + x / 8 : x;
  const int64_t i0 = (int64_t)blockIdx.y * BM, j0 = (int64_t)tile * BN;
  const int s = blockIdx.z;
  // slab sl of the part covers [k0 + sl kstep, + BK), loads stop at k1: a
  // contiguous part steps by BK through [cuts[s], cuts[s+1]); a strided part
  // (dealt tiles of width BK) steps by S BK from s BK up to K
  const bool strided = a.split_w != 0;
  const int64_t k0 = strided ? (int64_t)s * BK : a.cuts[s];
  const int64_t k1 = strided ? a.K : a.cuts[s + 1];
  const int64_t kstep = strided ? (int64_t)a.S * BK : BK;
  const int nslab = (k1 > k0) ? (int)((k1 - k0 + kstep - 1) / kstep) : 0;
  static_assert(CPR >= 8, "A rows of whole swizzle blocks");
  auto ldsA = [](int row, int c) { return row * CPR + (c ^ ((row >> 1) & 7)); };
  // rows of fewer than 8 chunks (BN < 64) are swizzled within the row
  auto ldsB = [](int k, int c) { return k * BROW + ((c ^ ((k & 3) << 1)) & (BROW - 1)); };

  u32x4 ra[D][ACH_T], rb[D][BCH_T];
  auto gload = [&](int sl, u32x4* xa, u32x4* xb) {
    const int64_t ks = k0 + (int64_t)sl * kstep;
#pragma unroll
    for (int t = 0; t < ACH_T; ++t) {
      const int q = tid + 256 * t, row = q / CPR, c = q % CPR;
      const int64_t gi = i0 + row, gk = ks + 8 * c;
      xa[t] = load_chunk<UN>((q < ACH) && (gi < a.M) && (gk < k1) && whole_a<UN>(a, gi, gk), a.A + gi * a.K + gk);
    }
#pragma unroll
    for (int t = 0; t < BCH_T; ++t) {
      const int q = tid + 256 * t, kr = q / BROW, c = q % BROW;
      const int64_t gk = ks + kr, gn = j0 + 8 * c;
      xb[t] = load_chunk<UN>((q < BCH) && (gk < k1) && (gn < a.N) && whole_b<UN>(a, gk, gn), a.B + gk * a.N + gn);
    }
  };
  auto lstore = [&](int buf, int sl, u32x4* xa, u32x4* xb) {
    uint16_t* As = As0 + buf * A_ELEMS;
    uint16_t* Bs = Bs0 + buf * B_ELEMS;
    if (UN && sl == nslab - 1) {   // contiguous parts only
      const int64_t ks = k0 + (int64_t)sl * kstep;
#pragma unroll
      for (int t = 0; t < ACH_T; ++t) {
        const int q = tid + 256 * t;
        if (q < ACH) xa[t] = last_a(a, xa[t], i0 + q / CPR, ks + 8 * (q % CPR), k1);
      }
#pragma unroll
      for (int t = 0; t < BCH_T; ++t) {
        const int q = tid + 256 * t;
        if (q < BCH) xb[t] = last_b(a, xb[t], ks + q / BROW, j0 + 8 * (q % BROW), k1);
      }
    }
#pragma unroll
    for (int t = 0; t < ACH_T; ++t) {
      const int q = tid + 256 * t;
      if (q < ACH) *(u32x4*)&As[8 * ldsA(q / CPR, q % CPR)] = xa[t];
    }
#pragma unroll
    for (int t = 0; t < BCH_T; ++t) {
      const int q = tid + 256 * t;
      if (q < BCH) *(u32x4*)&Bs[8 * ldsB(q / BROW, q % BROW)] = xb[t];
    }
  };
  floatx4 acc[TMS];
#pragma unroll
  for (int mi = 0; mi < TMS; ++mi) acc[mi] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) {
    if (wave >= NWC) return;
    const uint16_t* As = As0 + buf * A_ELEMS;
    const uint16_t* Bs = Bs0 + buf * B_ELEMS;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 32) {
      const int i = lane & 15, g = lane >> 4;
      const int n = 16 * wave + 4 * (i & 3);
      const int kr0 = kk + 8 * g + (i >> 2), kr1 = kr0 + 4;
      const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&Bs[8 * ldsB(kr0, n / 8) + (n & 7)]));
      const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&Bs[8 * ldsB(kr1, n / 8) + (n & 7)]));
      const shortx8 bfr = shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
      for (int mi = 0; mi < TMS; ++mi) {
        const shortx8 af = *(const shortx8*)&As[8 * ldsA(16 * mi + (lane & 15), kk / 8 + (lane >> 4))];
        acc[mi] = mfma16t<F16>(af, bfr, acc[mi]);
      }
    }
  };

  // Loads and LDS stores are issued unconditionally (a slab past the part
  // end reads the zero chunk), so that every path holds the same number of
  // loads in flight and the LDS store of slab s+1 waits only for its own
  // loads, not for the D-1 slabs behind it.  Only the MFMA work is skipped.
  static_for<0, D>([&](auto j) { gload(j, ra[j], rb[j]); });
  lstore(0, 0, ra[0], rb[0]);
  __syncthreads();
  for (int base = 0; base < nslab; base += D) {
    static_for<0, D>([&](auto u) {
      const int sl = base + u;
      if (sl < nslab) compute(sl & 1);
      gload(sl + D, ra[u], rb[u]);
      lstore((sl + 1) & 1, sl + 1, ra[(u + 1) % D], rb[(u + 1) % D]);
      __syncthreads();
    });
  }
  if (wave < NWC) {
#pragma unroll
    for (int mi = 0; mi < TMS; ++mi)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + 16 * mi + 4 * (lane >> 4) + r, j = j0 + 16 * wave + (lane & 15);
        if (i < a.M && j < a.N) finish(a, s, i, j, acc[mi][r]);
      }
  }
}

}  // namespace dg
