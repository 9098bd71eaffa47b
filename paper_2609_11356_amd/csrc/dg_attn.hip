// dg_attn.hip -- attention forward for gfx950 whose reduction order is the
// attention descriptor's (paper App. F), independent of the workgroup shape.
//
// Per query row the keys are walked in the descriptor's blocks (width w from
// key 0; under a causal mask the walk splits at the multiples of BLOCK_M:
// the unmasked stage is cut at the query block's start, the masked stage is
// walked from there).  At each block the row's running maximum m, denominator
// l and output row O (binary32) are updated:
//   s_t = RN32(q . k_t * qk_scale)   (+ -1e6 on a masked key above the diagonal)
//   mn = max(m, max_t s_t);  alpha = exp2(m - mn);  p_t = exp2(s_t - mn)
//   l = alpha l + rowsum(p)  (or one fma),  O = alpha O (+) P~ . V
// with P~ = p narrowed to bf16, exp2 the library's own (dg_device.h), the
// block's row sum a chain or the balanced tree over the block's positions,
// and the two matrix multiplications on v_mfma_f32_16x16x32_bf16: the score
// over the head dimension from +0 with the accumulator carried, P~ . V over
// the block's keys from the block start, with alpha O as the accumulator
// (pv_fma) or from +0 and then added.  The end: O / l, or O * (1 / l).
//
// Two kernels: attn_fwd_t (below, tree row sums accumulated in place) and
// attn_fwd, for the other orders, 16-row causal splits and some short walks over
// keys in blocks of 128 (rows_128): one wave per RW
// query rows (16 or 32: one or two 16-row MFMA tiles), NW waves per workgroup (the rows of a workgroup share one causal
// split: BLOCK_M is a multiple of RW NW).  Each block's K and V rows are in
// LDS (two buffers: the next block's rows are fetched into registers while
// the current block computes and stored at its end, one barrier per block;
// zero past the block end, so that a short block's missing positions have
// p = 0 and zero products, which leave every accumulator's bits as they
// are).  The wave keeps its Q fragments in registers and its S tile and O
// rows in MFMA accumulators (lane l: rows 4 (l / 16) + j, column l % 16 of a
// 16 x 16 tile).  Score column c of sub-tile st is key NST c + st of the
// block, so the first levels of the block's row-sum tree (key bits below
// NST) are adds within a lane and the last four are DPP lane steps; P~ goes
// through the wave's LDS area as [key][row] (four rows per 8-byte write) and
// comes back in operand layout through the transposing LDS read.
#include <type_traits>

#include "dg_attn_tile.h"
#include "dg_lanes.h"

namespace dg {

namespace {

// True when alpha[0..3] are 1 on every active lane (one ballot; uniform).
__device__ __forceinline__ bool all_one(const float* alpha) {
  const bool one = alpha[0] == 1.0f && alpha[1] == 1.0f && alpha[2] == 1.0f && alpha[3] == 1.0f;
  return __builtin_amdgcn_ballot_w64(!one) == 0;
}

__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

}  // namespace

template <int D, int W, int NW, int RW, bool TREE, bool PF, bool PVF>
__global__ __launch_bounds__(64 * NW) void attn_fwd(AttnArgs a) {
  constexpr int DC = D / 8, NST = W / 16, NDT = D / 16, QKS = D / 32, PVS = W / 32, RT = RW / 16;
  constexpr int LNST = NST == 2 ? 1 : NST == 4 ? 2 : 3;     // log2 NST
  constexpr int PG = RW / 4;                                  // 8-byte groups of a P~ row
  static_assert(D % 32 == 0 && W % 32 == 0 && DC >= 8 && (NST == 2 || NST == 4 || NST == 8), "whole steps");
  constexpr int CHUNKS = W * DC / (64 * NW);                  // K (and V) chunks per thread
  static_assert(!PF || W * DC % (64 * NW) == 0, "whole chunks per thread");
  constexpr int NBUF = PF ? 2 : 1;                            // LDS buffers of K and V
  __shared__ __attribute__((aligned(16))) uint16_t Ks[NBUF][W * D];
  __shared__ __attribute__((aligned(16))) uint16_t Vs[NBUF][W * D];
  __shared__ __attribute__((aligned(16))) uint16_t Ps[NW][W * RW];
  __shared__ float Fs[TREE ? 1 : NW][TREE ? 1 : RW * (W + 1)];   // the chained block sum

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lg = lane >> 4;
  // heads run fastest through the grid, and under a causal mask the query
  // blocks run from the last (the longest walk) to the first
  const int64_t h = blockIdx.x;
  const int64_t qb = a.causal ? (int64_t)gridDim.y - 1 - blockIdx.y : blockIdx.y;
  const int64_t r0 = qb * (RW * NW);
  const int64_t rw = r0 + RW * wave;
  const uint16_t* Qh = a.Q + h * a.Lq * D;
  const uint16_t* Kh = a.K + h * a.Lk * D;
  const uint16_t* Vh = a.V + h * a.Lk * D;

  // K row t: chunk c at c ^ (the row's lane index mod DC), so that the 16
  // rows one fragment read takes land on distinct 16-byte slots
  auto kofs = [](int t, int c) { return t * DC + (c ^ ((t >> LNST) & (DC - 1))); };
  auto vofs = [](int k, int c) {
    if constexpr (DC >= 16) return k * DC + (c ^ ((k & 3) << 1) ^ (((k >> 3) & 1) << 3));
    else return k * DC + (c ^ ((k & 3) << 1));
  };
  // P~ [key u][row r]: 8-byte group g of key row u at g ^ ((u >> LNST) mod PG)
  auto pofs = [](int u, int r) { return u * RW + 4 * ((r >> 2) ^ ((u >> LNST) & (PG - 1))) + (r & 3); };

  shortx8 qf[RT][QKS];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int64_t i = rw + 16 * rt + li;
#pragma unroll
    for (int k = 0; k < QKS; ++k)
      qf[rt][k] = i < a.Lq ? *(const shortx8*)&Qh[i * D + 32 * k + 8 * lg] : shortx8{0, 0, 0, 0, 0, 0, 0, 0};
  }

  float m[RT][4], l[RT][4];
  floatx4 O[RT][NDT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      m[rt][j] = -__builtin_inff();
      l[rt][j] = 0.f;
    }
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) O[rt][dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  // the walk: nb1 unmasked blocks of [0, end1) from key 0, then (causal) nb2
  // masked-stage blocks of [q0, q1) from q0
  int64_t end1 = a.Lk, q0 = 0, q1 = 0;
  if (a.causal) {
    q0 = r0 / a.q_block * a.q_block;
    q1 = q0 + a.q_block < a.Lk ? q0 + a.q_block : a.Lk;
    end1 = q0;
  }
  const int64_t nb1 = (end1 + W - 1) / W, nb = nb1 + (a.causal ? (q1 - q0 + W - 1) / W : 0);
  auto bounds = [&](int64_t b, int64_t* kb, int64_t* ke) {
    const bool st2 = b >= nb1;
    *kb = st2 ? q0 + (b - nb1) * W : b * W;
    const int64_t lim = st2 ? q1 : end1;
    *ke = *kb + W < lim ? *kb + W : lim;
  };
  u32x4 kr[PF ? CHUNKS : 1], vr[PF ? CHUNKS : 1];
  auto fetch = [&](int64_t b) {
    int64_t kb, ke;
    bounds(b, &kb, &ke);
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) {
      const int q = threadIdx.x + 64 * NW * u, t = q / DC, c = q % DC;
      kr[u] = vr[u] = u32x4{0u, 0u, 0u, 0u};
      if (kb + t < ke) {
        kr[u] = *(const u32x4*)&Kh[(kb + t) * D + 8 * c];
        vr[u] = *(const u32x4*)&Vh[(kb + t) * D + 8 * c];
      }
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int u = 0; u < CHUNKS; ++u) {
      const int q = threadIdx.x + 64 * NW * u, t = q / DC, c = q % DC;
      *(u32x4*)&Ks[buf][8 * kofs(t, c)] = kr[u];
      *(u32x4*)&Vs[buf][8 * vofs(t, c)] = vr[u];
    }
  };
  // without prefetch: the block straight from memory into the one buffer
  auto load_block = [&](int64_t b) {
    int64_t kb, ke;
    bounds(b, &kb, &ke);
    for (int q = threadIdx.x; q < W * DC; q += 64 * NW) {
      const int t = q / DC, c = q % DC;
      u32x4 kv = u32x4{0u, 0u, 0u, 0u}, vv = u32x4{0u, 0u, 0u, 0u};
      if (kb + t < ke) {
        kv = *(const u32x4*)&Kh[(kb + t) * D + 8 * c];
        vv = *(const u32x4*)&Vh[(kb + t) * D + 8 * c];
      }
      *(u32x4*)&Ks[0][8 * kofs(t, c)] = kv;
      *(u32x4*)&Vs[0][8 * vofs(t, c)] = vv;
    }
  };
  if constexpr (PF) {
    if (nb > 0) {
      fetch(0);
      stash(0);
    }
  }

  for (int64_t b = 0; b < nb; ++b) {
    const int cur = PF ? (int)(b & 1) : 0;
    int64_t kb, ke;
    bounds(b, &kb, &ke);
    const bool masked = b >= nb1;
    const bool edge = masked || ke - kb < W;
    __syncthreads();
    if constexpr (PF) {
      if (b + 1 < nb) fetch(b + 1);
    } else {
      load_block(b);
      __syncthreads();
    }
    const uint16_t* K_ = Ks[cur];
    const uint16_t* V_ = Vs[cur];

    // scores: RW rows x W keys (column c of sub-tile st: key NST c + st), the
    // head dimension in increasing steps of 32 from +0; then scaled
    floatx4 S[RT][NST];
#pragma unroll
    for (int st = 0; st < NST; ++st) {
      shortx8 kf[QKS];
#pragma unroll
      for (int k = 0; k < QKS; ++k) kf[k] = *(const shortx8*)&K_[8 * kofs(NST * li + st, 4 * k + lg)];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < QKS; ++k) acc = mfma(qf[rt][k], kf[k], acc);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = acc[j] * a.qk_scale;
        S[rt][st] = acc;
      }
    }
    // positions past the block end drop out (-inf), masked keys get -1e6
    if (edge) {
#pragma unroll
      for (int st = 0; st < NST; ++st) {
        const int64_t t = kb + NST * li + st;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int64_t i = rw + 16 * rt + 4 * lg + j;
            float v = S[rt][st][j];
            if (t >= ke) v = -__builtin_inff();
            else if (masked && t > i) v = v + -1.0e6f;
            S[rt][st][j] = v;
          }
      }
    }

#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float alpha[4], rs[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float bm = S[rt][0][j];
#pragma unroll
        for (int st = 1; st < NST; ++st) bm = __builtin_fmaxf(bm, S[rt][st][j]);
        bm = max_lanes<4>(bm);
        const float mn = __builtin_fmaxf(m[rt][j], bm);
        alpha[j] = exp2_f32(m[rt][j] - mn);
        m[rt][j] = mn;
#pragma unroll
        for (int st = 0; st < NST; ++st) S[rt][st][j] = exp2_f32(S[rt][st][j] - mn);
      }
      if constexpr (TREE) {
        // the perfect tree over the block's positions in key order: key bits
        // below NST within the lane, then the 16 lanes of the row group
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float v[NST];
#pragma unroll
          for (int st = 0; st < NST; ++st) v[st] = S[rt][st][j];
#pragma unroll
          for (int w2 = 1; w2 < NST; w2 <<= 1)
#pragma unroll
            for (int st = 0; st < NST; st += 2 * w2) v[st] = v[st] + v[st + w2];
          rs[j] = tree_sum_lanes<4>(v[0]);
        }
      } else {
        // the chain in key order through the wave's LDS area
        float* F = Fs[wave];
#pragma unroll
        for (int st = 0; st < NST; ++st)
#pragma unroll
          for (int j = 0; j < 4; ++j) F[(16 * rt + 4 * lg + j) * (W + 1) + NST * li + st] = S[rt][st][j];
        lds_wait();
        if (lane < 16) {
          const float* row = &F[(16 * rt + lane) * (W + 1)];
          float x = row[0];
          for (int u = 1; u < W; ++u) x = x + row[u];
          F[(16 * rt + lane) * (W + 1) + W] = x;
        }
        lds_wait();
#pragma unroll
        for (int j = 0; j < 4; ++j) rs[j] = F[(16 * rt + 4 * lg + j) * (W + 1) + W];
        lds_wait();
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) l[rt][j] = a.l_fma ? __builtin_fmaf(alpha[j], l[rt][j], rs[j]) : alpha[j] * l[rt][j] + rs[j];

      // P~ = p narrowed to bf16 into the wave's [key][row] area, four rows per write
      uint16_t* P = Ps[wave];
#pragma unroll
      for (int st = 0; st < NST; ++st) {
        const int u = NST * li + st;
        const uint32_t lo = f32x2_bf16x2(S[rt][st][0], S[rt][st][1]), hi = f32x2_bf16x2(S[rt][st][2], S[rt][st][3]);
        *(uint2*)&P[pofs(u, 16 * rt + 4 * lg)] = uint2{lo, hi};
      }
      // rescale the output rows (skipped when every row of the wave keeps its
      // maximum: alpha = 1 and 1 x O = O exactly)
      if (!all_one(alpha))
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
          for (int j = 0; j < 4; ++j) O[rt][dt][j] = alpha[j] * O[rt][dt][j];
    }
    lds_wait();

    // O = alpha O (+) P~ . V over the block's keys from its start, for each
    // output element the steps of 32 keys in increasing order
    const uint16_t* P = Ps[wave];
    shortx8 pf[RT][PVS];
#pragma unroll
    for (int k = 0; k < PVS; ++k)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int n = 16 * rt + 4 * (li & 3);
        const int u0 = 32 * k + 8 * lg + (li >> 2), u1 = u0 + 4;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&P[pofs(u0, n)]));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&P[pofs(u1, n)]));
        pf[rt][k] = shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      }
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
      floatx4 acc[RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[rt] = PVF ? O[rt][dt] : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < PVS; ++k) {
        const int n = 16 * dt + 4 * (li & 3);
        const int kr0 = 32 * k + 8 * lg + (li >> 2), kr1 = kr0 + 4;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&V_[8 * vofs(kr0, n >> 3) + (n & 7)]));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&V_[8 * vofs(kr1, n >> 3) + (n & 7)]));
        const shortx8 vf = shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt] = mfma(pf[rt][k], vf, acc[rt]);
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        if constexpr (PVF) O[rt][dt] = acc[rt];
        else
#pragma unroll
          for (int j = 0; j < 4; ++j) O[rt][dt][j] = O[rt][dt][j] + acc[rt][j];
      }
    }
    if constexpr (PF) {
      if (b + 1 < nb) stash(cur ^ 1);
    }
  }

  // the final division (or reciprocal and products), then the output type
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float r[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = 1.0f / l[rt][j];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t i = rw + 16 * rt + 4 * lg + j;
        if (i >= a.Lq) continue;
        const float y = a.final_recip ? O[rt][dt][j] * r[j] : O[rt][dt][j] / l[rt][j];
        const int64_t o = (h * a.Lq + i) * D + 16 * dt + li;
        if (a.out_bf16) ((uint16_t*)a.O)[o] = f32_bf16(y);
        else ((float*)a.O)[o] = y;
      }
  }
}

// ------------------------------------------------ transposed score tiles
//
// The tree row sum with P V accumulated in place (pv_fma), RW = 32 or 16
// query rows per wave on v_mfma_f32_32x32x16_bf16 or 16x16x32 (chunks of 8 k
// either way, so the same bits).  The tiles are computed transposed --
// S^T = K Q^T, O^T += V^T P~^T -- so that a lane owns one query row (l % RW;
// G = l / RW names its share of the keys):
//   * the maximum, the row sum and the rescale are in-lane work plus one
//     (RW 32) or two exchanges between lane groups, and alpha is one
//     exponential per row, not one per row and lane group;
//   * the rows of a K tile are taken in an order (kmap) that leaves lane l
//     with keys KS kk + 8 G + 0..7 of every KS-key step kk: exactly its
//     operand of the P~ V instruction, so P~ never leaves the registers (the
//     kernel above passes it through LDS);
//   * with RW = 32 each K and V fragment read from LDS serves 32 rows.
// The row-sum tree: 8 keys in the lane, the lane groups by v_permlane swaps,
// then the steps' nodes in key order.
//
// Bound: VALU.  A score takes 16 instructions (scale, half a maximum,
// subtract, twelve for 2^x, tree add, half a conversion) at four cycles a
// wave.  So the products run under them: while step kk's exponentials are
// computed, the matrix cores work on P~ V of step kk - 1 and on K Q^T of the
// next block (K runs a block ahead of V in LDS), and a second workgroup per
// CU fills what is left.
//
// The K and V rows of a key block go from memory straight into LDS
// (buffer_load ... lds), a block ahead in a second pair of arrays; the arrays
// are separate variables so that the compiler waits for a pair's loads only.
template <int D, int W, int NW, int RW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(W * D * RW > 64 * 128 * 32 ? 1 : 2))) void
attn_fwd_t(AttnArgs a) {
  constexpr int DC = D / 8, KS = RW == 32 ? 16 : 32;       // chunks of a row; keys per P V step
  constexpr int NK = W / KS, NP = W * RW / 64;             // steps; scores per lane
  constexpr int QKS = D / KS, ND = D / RW, NT = W / RW;    // head-dimension steps, O and S tiles
  constexpr int TR = RW == 32 ? 16 : 4;                    // registers per tile
  constexpr int NQ = NT * QKS;                             // score instructions per block
  constexpr int NLD = W * DC / (64 * NW);                  // K (and V) loads per wave and block, 1 KB each
  static_assert(W * DC % (64 * NW) == 0, "whole loads per wave");
  typedef std::conditional_t<RW == 32, floatx16, floatx4> tile_t;
  __shared__ __attribute__((aligned(1024))) uint16_t K0[W * D];
  __shared__ __attribute__((aligned(1024))) uint16_t V0[W * D];
  __shared__ __attribute__((aligned(1024))) uint16_t K1[W * D];
  __shared__ __attribute__((aligned(1024))) uint16_t V1[W * D];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & (RW - 1), G = lane / RW;
  const int64_t h = blockIdx.x;
  const int64_t qb = a.causal ? (int64_t)gridDim.y - 1 - blockIdx.y : blockIdx.y;
  const int64_t r0 = qb * (RW * NW);
  const int64_t row = r0 + RW * wave + li;       // the lane's query row
  const uint16_t* Qh = a.Q + h * a.Lq * D;
  // every byte offset within a head's K and V fits 31 bits (the host checks)
  const int rec = (int)(a.Lk * D * 2);
  const __amdgpu_buffer_rsrc_t rK = __builtin_amdgcn_make_buffer_rsrc((void*)(a.K + h * a.Lk * D), (short)0, rec, 0x00020000);
  const __amdgpu_buffer_rsrc_t rV = __builtin_amdgcn_make_buffer_rsrc((void*)(a.V + h * a.Lk * D), (short)0, rec, 0x00020000);

  // the lane's fragment addresses (elements; tiles and key steps add constants,
  // which leave the swizzles as they are)
  const int kmap = key_of_row<RW>(li);
  const int vi = lane & 15, vrow = (RW == 32 ? 8 * G : 8 * (lane >> 4)) + (vi >> 2);
  const int vcol = (RW == 32 ? 16 * ((lane >> 4) & 1) : 0) + 4 * (vi & 3);
  constexpr int CPS = KS / 8;                    // chunks per head-dimension step
  int kad[QKS], vad[ND];
#pragma unroll
  for (int k = 0; k < QKS; ++k) kad[k] = 8 * (kmap * DC + ((CPS * k + G) ^ k_swz<RW, DC>(kmap)));
#pragma unroll
  for (int dt = 0; dt < ND; ++dt) vad[dt] = 8 * (vrow * DC + (((RW * dt + vcol) >> 3) ^ v_swz<RW, DC>(vrow))) + (vcol & 7);
  // first key of tile T relative to the lane's kmap
  auto tile_key = [](int T) { return RW == 32 ? 32 * T : 32 * (T >> 1) + 4 * (T & 1); };
  // score register i of the lane: the key (relative to 8 G)
  auto key_of = [](int i) { return KS * (i >> 3) + (i & 7); };

  shortx8 qf[QKS];
#pragma unroll
  for (int k = 0; k < QKS; ++k)
    qf[k] = row < a.Lq ? *(const shortx8*)&Qh[row * D + KS * k + 8 * G] : shortx8{0, 0, 0, 0, 0, 0, 0, 0};

  float m = -__builtin_inff(), l = 0.f;
  tile_t O[ND], Sn[NT];
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int i = 0; i < TR; ++i) O[dt][i] = 0.f;

  int end1 = (int)a.Lk, q0 = 0, q1 = 0;
  if (a.causal) {
    q0 = (int)(r0 / a.q_block * a.q_block);
    q1 = q0 + a.q_block < a.Lk ? q0 + a.q_block : (int)a.Lk;
    end1 = q0;
  }
  const int nb1 = (end1 + W - 1) / W, nb = nb1 + (a.causal ? (q1 - q0 + W - 1) / W : 0);
  auto bounds = [&](int b, int* kb, int* ke) {
    const bool st2 = b >= nb1;
    *kb = st2 ? q0 + (b - nb1) * W : b * W;
    const int lim = st2 ? q1 : end1;
    *ke = *kb + W < lim ? *kb + W : lim;
  };
  // load i of the wave fills LDS chunks 64 (NLD wave + i) + lane; the lane
  // fetches the chunk that belongs there (rows past the block end: zeros)
  auto fetch = [&](bool v, uint16_t* dst, int b) {
    if (b >= nb) return;
    int kb, ke;
    bounds(b, &kb, &ke);
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int q = 64 * (NLD * wave + i) + lane, t = q / DC, c = (q % DC) ^ (v ? v_swz<RW, DC>(t) : k_swz<RW, DC>(t));
      const uint32_t off = kb + t < ke ? (uint32_t)((t * DC + c) * 16) : 0x80000000u;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(v ? rV : rK, (lds_void)(dst + 512 * (NLD * wave + i)), 16, off,
                                               kb * D * 2, 0, 0);
    }
  };
  // score instruction u of a block: head-dimension step u % QKS of tile u / QKS
  auto score = [&](const uint16_t* K_, int u) {
    const int T = u / QKS, k = u % QKS;
    if (k == 0)
#pragma unroll
      for (int i = 0; i < TR; ++i) Sn[T][i] = 0.f;
    mfma_to(Sn[T], *(const shortx8*)&K_[kad[k] + tile_key(T) * D], qf[k]);
  };

  // One key block: its scores in Sn, its V rows in V_; the next block's K rows
  // in Kn (whose scores are left in Sn; past the last block they are not used).
  auto block = [&](int b, const uint16_t* V_, const uint16_t* Kn) {
    int kb, ke;
    bounds(b, &kb, &ke);
    const bool masked = b >= nb1;
    float S[NP];
#pragma unroll
    for (int T = 0; T < NT; ++T)
#pragma unroll
      for (int i = 0; i < TR; ++i) S[TR * T + i] = Sn[T][i] * a.qk_scale;
    // positions past the block end drop out (-inf), masked keys get -1e6
    if (masked || ke - kb < W) {
      const int left = ke - kb - 8 * G, diag = masked ? (int)row - kb - 8 * G : W;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        float v = S[i];
        if (key_of(i) >= left) v = -__builtin_inff();
        else if (key_of(i) > diag) v = v + -1.0e6f;
        S[i] = v;
      }
    }
    float bm = S[0];
#pragma unroll
    for (int i = 1; i < NP; ++i) bm = __builtin_fmaxf(bm, S[i]);
    float bo = bm;
    if constexpr (RW == 16) {
      rows_swap(bm, bo);
      bm = __builtin_fmaxf(bm, bo);
      bo = bm;
    }
    halves_swap(bm, bo);
    const float mn = __builtin_fmaxf(m, __builtin_fmaxf(bm, bo));
    const float alpha = exp2_nonpos(m - mn);
    m = mn;
    // rescale the output rows (skipped when every row of the wave keeps its
    // maximum: alpha = 1 and 1 x O = O exactly)
    if (__builtin_amdgcn_ballot_w64(!(alpha == 1.0f)) != 0) {
#pragma unroll
      for (int dt = 0; dt < ND; ++dt)
#pragma unroll
        for (int i = 0; i < TR; ++i) O[dt][i] = alpha * O[dt][i];
    }
    float n8[NK];
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      __builtin_amdgcn_sched_barrier(0);
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = exp2_nonpos(S[8 * kk + e] - mn);
      // P~ = p narrowed to bf16, already in operand layout
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = f32x2_bf16x2(v[2 * e], v[2 * e + 1]);
      const shortx8 pf = __builtin_bit_cast(shortx8, w);
      // the perfect tree over the block's keys in order
#pragma unroll
      for (int x = 1; x < 8; x <<= 1)
#pragma unroll
        for (int e = 0; e < 8; e += 2 * x) v[e] = v[e] + v[e + x];
      n8[kk] = v[0];
      // the next block's scores, then O^T = alpha O^T (+) V^T P~^T: for each
      // output the steps of KS keys in increasing order
#pragma unroll
      for (int u = kk * NQ / NK; u < (kk + 1) * NQ / NK; ++u) score(Kn, u);
#pragma unroll
      for (int dt = 0; dt < ND; ++dt) {
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&V_[vad[dt] + KS * kk * D]));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(&V_[vad[dt] + (KS * kk + 4) * D]));
        mfma_to(O[dt], shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]}, pf);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (RW == 32) {
      // one swap turns two values spread over the halves into their two sums:
      // 2^j values -> 2^(j-1) registers (one per half), down to the root
#pragma unroll
      for (int c = NK; c > 1; c >>= 1)
#pragma unroll
        for (int e = 0; e < c / 2; ++e) {
          float x = n8[2 * e], y = n8[2 * e + 1];
          halves_swap(x, y);
          n8[e] = x + y;
        }
      float y = n8[0];
      halves_swap(n8[0], y);
      n8[0] = n8[0] + y;
    } else {
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        float y = n8[kk];
        rows_swap(n8[kk], y);
        n8[kk] = n8[kk] + y;
        y = n8[kk];
        halves_swap(n8[kk], y);
        n8[kk] = n8[kk] + y;
      }
#pragma unroll
      for (int x = 1; x < NK; x <<= 1)
#pragma unroll
        for (int kk = 0; kk < NK; kk += 2 * x) n8[kk] = n8[kk] + n8[kk + x];
    }
    l = a.l_fma ? __builtin_fmaf(alpha, l, n8[0]) : alpha * l + n8[0];
  };

  // A wave's own loads have landed once its count is zero; after the barrier
  // that follows, everybody's have, and the K pair of block b and the V pair of
  // block b - 1 are free for the loads of blocks b + 2 and b + 1.
  auto turn = [&]() {
    __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
    barrier_nofence();
  };
  fetch(false, K0, 0);
  fetch(true, V0, 0);
  turn();
  fetch(false, K1, 1);
#pragma unroll
  for (int u = 0; u < NQ; ++u) score(K0, u);
  for (int b = 0; b < nb; b += 2) {
    turn();
    fetch(false, K0, b + 2);
    fetch(true, V1, b + 1);
    block(b, V0, K1);
    turn();
    fetch(false, K1, b + 3);
    fetch(true, V0, b + 2);
    if (b + 1 < nb) block(b + 1, V1, K0);
  }

  // the final division (or reciprocal and products), then the output type;
  // register i of tile dt holds column RW dt + 8 (i / 4) + 4 G + i % 4 (RW 32)
  // or 16 dt + 4 G + i (RW 16)
  if (row >= a.Lq) return;
  const float r = 1.0f / l;
#pragma unroll
  for (int dt = 0; dt < ND; ++dt)
#pragma unroll
    for (int c = 0; c < TR / 4; ++c) {
      float y[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = a.final_recip ? O[dt][4 * c + e] * r : O[dt][4 * c + e] / l;
      const int64_t o = (h * a.Lq + row) * D + RW * dt + 8 * c + 4 * G;
      if (a.out_bf16) *(uint2*)&((uint16_t*)a.O)[o] = uint2{f32x2_bf16x2(y[0], y[1]), f32x2_bf16x2(y[2], y[3])};
      else *(float4*)&((float*)a.O)[o] = float4{y[0], y[1], y[2], y[3]};
    }
}

namespace {

template <int D, int W, int NW, int RW, bool PF>
hipError_t launch_one(const AttnArgs& a, hipStream_t st) {
  constexpr int rows = NW * RW;
  dim3 grid((unsigned)a.H, (unsigned)((a.Lq + rows - 1) / rows));
  const dim3 blk(64 * NW);
  if (a.block_tree) {
    if (a.pv_fma) hipLaunchKernelGGL((attn_fwd<D, W, NW, RW, true, PF, true>), grid, blk, 0, st, a);
    else hipLaunchKernelGGL((attn_fwd<D, W, NW, RW, true, PF, false>), grid, blk, 0, st, a);
  } else {
    if (a.pv_fma) hipLaunchKernelGGL((attn_fwd<D, W, NW, RW, false, PF, true>), grid, blk, 0, st, a);
    else hipLaunchKernelGGL((attn_fwd<D, W, NW, RW, false, PF, false>), grid, blk, 0, st, a);
  }
  return hipGetLastError();
}

template <int D, int W, int NW, int RW>
hipError_t launch_t(const AttnArgs& a, hipStream_t st) {
  constexpr int rows = RW * NW;
  dim3 grid((unsigned)a.H, (unsigned)((a.Lq + rows - 1) / rows));
  hipLaunchKernelGGL((attn_fwd_t<D, W, NW, RW>), grid, dim3(64 * NW), 0, st, a);
  return hipGetLastError();
}

// Rows per wave of attn_fwd_t, or 0 where attn_fwd is the faster one, for
// d = 128 and keys in blocks of 128 (speed only): attn_fwd_t's 128 KB of LDS
// leave one workgroup per CU, attn_fwd's 80 KB two, so its overlap within a
// workgroup has to make up for the second one.  Measured on MI355X, attn_fwd /
// attn_fwd_t, operands from HBM, H heads of Lq x Lk:
//   128-row workgroups (32-row waves) need more than one key block (2000 x 40
//   0.76, 500 x 33 0.8, 128 x 128 0.93 to 1.04, 2000 x 200 0.96 to 1.09, 512 x
//   512 1.3), and, where the last of them is half empty, keys enough for that
//   too: 129 x 129 0.77, 257 x 257 0.9, 300 x 900 1.1 to 1.4, 130 x 1000 1.25
//   (unmasked; causal at most 1.2, so half as many keys again: 400 x 400 0.97);
//   64-row workgroups gain while each has a CU (H 256, 64 x 64 1.24; H 64,
//   256 x 256 1.54), while two rounds of them stand against one of attn_fwd
//   from two or three blocks of keys (H 384, 64 x 64 0.83; H 64, 257 x 257
//   0.93, 300 x 900 1.17; causal H 128, 129 x 129 0.87, 256 x 256 1.10), and in
//   more rounds on long keys only (causal H 512, 256 x 256 0.80, 640 x 640
//   0.92; H 203, 1500 x 1500 1.02).
int rows_128(const AttnArgs& a, bool rows32) {
  constexpr int64_t ncu = 256;
  const int64_t r64 = (a.Lq + 63) / 64, wg = a.H * r64;
  const int64_t half = r64 % 2 ? (a.causal ? 2304 : 1536) / (r64 + 1) : 0;
  if (rows32 && a.Lk > 128 + half) return 32;
  if (wg <= ncu || a.Lk > 1024 || (wg <= 2 * ncu && a.Lk >= (a.causal ? 192 : 320))) return 16;
  return 0;
}

// Workgroup shape of attn_fwd (speed only): 16-row waves (registers), eight of
// them with the next block prefetched into a second buffer when the causal
// split allows 128-row workgroups (four when it allows 64), else fewer waves
// loading each block as it comes.
// Measured on MI355X, attn_fwd -> attn_fwd_t: 32 heads x 4096 x 128, blocks of
// 64, 653 -> 383 us unmasked (717 TFLOP/s; 86 % of the VALU's cycles while a
// CU is busy), 349 -> 219 us causal; blocks of 32 453 -> 247, of 128 401 -> 284
// (causal); d = 64 219 -> 150; 16 heads x 1000 x 128 causal, 16-row waves, 41 ->
// 26 (32-row waves: 45).
template <int D, int W>
hipError_t launch_dw(const AttnArgs& a, hipStream_t st) {
  const int64_t bm = a.causal ? a.q_block : 128;
  // tree row sums accumulated in place (a head's K and V within 31-bit
  // offsets): 32-row waves once they fill the chip's 1024 SIMDs, else 16-row
  // ones, whose blocks take half the time
  if (a.block_tree && a.pv_fma && a.Lk * D * 2 <= 0x7fffffff) {
    // (and where 128-key blocks leave room for few workgroups, rows enough that
    // half of the waves aren't idle: d = 64, H 512, 64 x 64 12.8 -> 9.5 us)
    const bool full = a.H * ((a.Lq + 31) / 32) >= 1024 && (W < 128 || a.Lq > 64);
    int rows = bm % 128 == 0 && full ? 32 : 16;
    if (W == 128 && D == 128 && bm % 64 == 0) rows = rows_128(a, rows == 32);
    if (rows == 32) return launch_t<D, W, 4, 32>(a, st);
    if (rows == 16 && bm % 64 == 0) return launch_t<D, W, 4, 16>(a, st);
    if (bm % 64 && bm % 32 == 0) return launch_t<D, W, 2, 16>(a, st);
  }
  if constexpr (W == 128) {
    if (bm % 64 == 0) return launch_one<D, W, 4, 16, false>(a, st);
    return launch_one<D, W, 1, 16, false>(a, st);
  } else {
    // prefetch needs whole 16-byte chunks of the block per thread
    constexpr bool pf8 = W * (D / 8) % 512 == 0, pf4 = W * (D / 8) % 256 == 0;
    if (bm % 128 == 0) return launch_one<D, W, 8, 16, pf8>(a, st);
    if (bm % 64 == 0) return launch_one<D, W, 4, 16, pf4>(a, st);
    if (bm % 32 == 0) return launch_one<D, W, 2, 16, false>(a, st);
    return launch_one<D, W, 1, 16, false>(a, st);
  }
}

}  // namespace

bool attn_supported(int64_t d, int key_block) {
  return (d == 64 || d == 128) && (key_block == 32 || key_block == 64 || key_block == 128);
}

hipError_t launch_attention(const AttnArgs& a, int64_t d, int key_block, hipStream_t st) {
  if (d == 64) {
    if (key_block == 32) return launch_dw<64, 32>(a, st);
    if (key_block == 64) return launch_dw<64, 64>(a, st);
    return launch_dw<64, 128>(a, st);
  }
  if (key_block == 32) return launch_dw<128, 32>(a, st);
  if (key_block == 64) return launch_dw<128, 64>(a, st);
  return launch_dw<128, 128>(a, st);
}

}  // namespace dg
