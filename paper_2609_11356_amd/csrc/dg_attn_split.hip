// dg_attn_split.hip -- attention for few query rows (decoding, short cross
// attention): the key blocks of a row spread over the chip.
//
// With few rows the one-launch kernels (dg_attn.hip) walk the key blocks one
// after another on a handful of workgroups, and each block costs a memory
// latency (32 heads x 1 x 4001 x 128: 84 us for 66 MB).  The order ties only
// cheap things along the walk -- the running maximum, the denominator, and
// the accumulator chain of O -- so the rest is done for all blocks at once,
// in three launches through a workspace of one record per (16-row tile, key
// block):
//   attn_split_scores  a wave per record: the block's scaled (and masked)
//                      scores and their row maxima;
//   attn_split_probs   a wave per record: the running maximum before and
//                      after the block (a maximum over the earlier records'
//                      maxima: exact, in any order), alpha, the narrowed
//                      probabilities (over the scores' place) and the block's
//                      row sum;
//   attn_split_out     a wave per tile and 16 output columns: O = alpha O, the
//                      P~ V steps of the block, l's update, block by block;
//                      the records and V's columns stream through a ring of
//                      LDS slots, RD blocks ahead.
// Every value takes the steps of the one-launch kernels, so the bits are
// theirs.  The layouts are those of transposed score tiles with 16 rows
// (dg_attn.hip): lane l owns query row l % 16 and keys 32 kk + 8 (l / 16) +
// 0..7, and P~ is stored as the operand registers it will be loaded into.
//
// Bound: the K and V streams (HBM), then launches.  Measured on MI355X, one
// launch -> split: see attn_split_ok.
#include "dg_attn_tile.h"

namespace dg {

namespace {

// A record: S (or P~ over it), then m_block, alpha and row sum of 16 rows each.
template <int W>
constexpr int rec_floats() { return 16 * W + 48; }

struct SplitArgs {
  AttnArgs a;
  float* ws;
  int32_t tiles, nb_max;        // 16-row tiles of all heads; records per tile
};

// The walk of the tile's rows: nb blocks, block b covering keys [kb, ke).
template <int W>
struct Walk {
  int end1, q0, q1, nb1, nb;
  __device__ __forceinline__ Walk(const AttnArgs& a, int64_t r0) {
    end1 = (int)a.Lk;
    q0 = q1 = 0;
    if (a.causal) {
      q0 = (int)(r0 / a.q_block * a.q_block);
      q1 = q0 + a.q_block < a.Lk ? q0 + a.q_block : (int)a.Lk;
      end1 = q0;
    }
    nb1 = (end1 + W - 1) / W;
    nb = nb1 + (a.causal ? (q1 - q0 + W - 1) / W : 0);
  }
  __device__ __forceinline__ void block(int b, int* kb, int* ke) const {
    const bool st2 = b >= nb1;
    *kb = st2 ? q0 + (b - nb1) * W : b * W;
    const int lim = st2 ? q1 : end1;
    *ke = *kb + W < lim ? *kb + W : lim;
  }
};

// Maximum over the four lane groups that share a query row.
__device__ __forceinline__ float groups_max(float x) {
  float y = x;
  rows_swap(x, y);
  x = __builtin_fmaxf(x, y);
  y = x;
  halves_swap(x, y);
  return __builtin_fmaxf(x, y);
}

}  // namespace

template <int D, int W>
__global__ __launch_bounds__(256) void attn_split_scores(SplitArgs s) {
  constexpr int QKS = D / 32, NT = W / 16, NP = W / 4;
  const AttnArgs& a = s.a;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x * 4 + wave, tile = blockIdx.y;
  const int qt = (int)((a.Lq + 15) / 16);
  const int64_t h = tile / qt, r0 = (int64_t)(tile % qt) * 16;
  const Walk<W> walk(a, r0);
  if (b >= walk.nb) return;
  int kb, ke;
  walk.block(b, &kb, &ke);
  const int li = lane & 15, G = lane >> 4, kmap = key_of_row<16>(li);
  const int64_t row = r0 + li;
  const shortx8 none = {0, 0, 0, 0, 0, 0, 0, 0};
  const uint16_t* Kh = a.K + h * a.Lk * D;
  shortx8 kf[NT][QKS], qf[QKS];
#pragma unroll
  for (int T = 0; T < NT; ++T) {
    const int key = kb + kmap + 32 * (T >> 1) + 4 * (T & 1);
#pragma unroll
    for (int k = 0; k < QKS; ++k)
      kf[T][k] = key < ke ? *(const shortx8*)&Kh[(int64_t)key * D + 32 * k + 8 * G] : none;
  }
#pragma unroll
  for (int k = 0; k < QKS; ++k)
    qf[k] = row < a.Lq ? *(const shortx8*)&a.Q[(h * a.Lq + row) * D + 32 * k + 8 * G] : none;
  float S[NP];
#pragma unroll
  for (int T = 0; T < NT; ++T) {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < QKS; ++k) mfma_to(acc, kf[T][k], qf[k]);
#pragma unroll
    for (int i = 0; i < 4; ++i) S[4 * T + i] = acc[i] * a.qk_scale;
  }
  const bool masked = b >= walk.nb1;
  if (masked || ke - kb < W) {
    const int left = ke - kb - 8 * G, diag = masked ? (int)row - kb - 8 * G : W;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int t = 32 * (i >> 3) + (i & 7);
      float v = S[i];
      if (t >= left) v = -__builtin_inff();
      else if (t > diag) v = v + -1.0e6f;
      S[i] = v;
    }
  }
  float bm = S[0];
#pragma unroll
  for (int i = 1; i < NP; ++i) bm = __builtin_fmaxf(bm, S[i]);
  bm = groups_max(bm);
  float* rec = s.ws + ((int64_t)tile * s.nb_max + b) * rec_floats<W>();
#pragma unroll
  for (int i = 0; i < NP; ++i) rec[64 * i + lane] = S[i];
  if (G == 0) rec[16 * W + li] = bm;
}

template <int W>
__global__ __launch_bounds__(256) void attn_split_probs(SplitArgs s) {
  constexpr int NK = W / 32, NP = W / 4, RF = rec_floats<W>();
  const AttnArgs& a = s.a;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x * 4 + wave, tile = blockIdx.y;
  const int64_t r0 = (int64_t)(tile % (int)((a.Lq + 15) / 16)) * 16;
  const Walk<W> walk(a, r0);
  if (b >= walk.nb) return;
  const int li = lane & 15, G = lane >> 4;
  float* tws = s.ws + (int64_t)tile * s.nb_max * RF;
  float* rec = tws + (int64_t)b * RF;
  float S[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) S[i] = rec[64 * i + lane];
  // the running maximum before the block: lane group G takes every fourth record
  float m = -__builtin_inff();
  // (eight loads in flight; past b - 1 the last one again)
  for (int c = G; c < b; c += 32) {
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = tws[(int64_t)(c + 4 * u < b ? c + 4 * u : b - 1) * RF + 16 * W + li];
#pragma unroll
    for (int u = 0; u < 8; ++u) m = __builtin_fmaxf(m, x[u]);
  }
  m = groups_max(m);
  const float mn = __builtin_fmaxf(m, rec[16 * W + li]);
  const float alpha = exp2_nonpos(m - mn);
  float n8[NK];
  u32x4 pw[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = exp2_nonpos(S[8 * kk + e] - mn);
#pragma unroll
    for (int e = 0; e < 4; ++e) pw[kk][e] = f32x2_bf16x2(v[2 * e], v[2 * e + 1]);
#pragma unroll
    for (int x = 1; x < 8; x <<= 1)
#pragma unroll
      for (int e = 0; e < 8; e += 2 * x) v[e] = v[e] + v[e + x];
    float y = v[0];
    rows_swap(v[0], y);
    v[0] = v[0] + y;
    y = v[0];
    halves_swap(v[0], y);
    n8[kk] = v[0] + y;
  }
#pragma unroll
  for (int x = 1; x < NK; x <<= 1)
#pragma unroll
    for (int kk = 0; kk < NK; kk += 2 * x) n8[kk] = n8[kk] + n8[kk + x];
  // every score of the record is in registers: P~ takes their place
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) *(u32x4*)&rec[256 * kk + 4 * lane] = pw[kk];
  if (G == 0) {
    rec[16 * W + 16 + li] = alpha;
    rec[16 * W + 32 + li] = n8[0];
  }
}

// Slot S of the ring: V's 16 columns, then P~ (separate arrays, so that a read
// waits for its own slot's loads only).
typedef __attribute__((address_space(3))) char* lds_char;
template <int W, int S>
__device__ __forceinline__ char* split_slot() {
  __shared__ __attribute__((aligned(1024))) char L[64 * W];
  return L;
}

// RD blocks in flight; a block is W / 32 loads of V's 16 columns (1 KB each,
// 32 keys), W / 32 of P~ and one each of alpha and the row sum.
// A wave alone on its SIMD issues one instruction every four cycles or more,
// so the loop is bound by instructions, not only by its chain: unmasked, the
// blocks past the end need no test (their V rows and records lie past the
// resources' ends and read as zeros: the range check counts the scalar offset
// too, as measured within one allocation), and every address is a lane
// constant plus one scalar that advances a block.
template <int D, int W, int RD, bool CAUSAL>
__global__ __launch_bounds__(64) void attn_split_out(SplitArgs s) {
  constexpr int NK = W / 32, ND = D / 16, RF = rec_floats<W>(), PER = 2 * NK + 2;
  static_assert(RD % 2 == 0 && (RD - 1) * PER <= 63, "the waits fit the load counter");
  const AttnArgs& a = s.a;
  const int lane = threadIdx.x, li = lane & 15, G = lane >> 4;
  // workgroup w runs on XCD w % 8: a tile's column blocks, which share V's
  // 128-byte lines, stay on one XCD
  const int w = blockIdx.x, tile = (w % 8) + 8 * (w / 8 / ND), dt = w / 8 % ND;
  if (tile >= s.tiles) return;
  const int qt = (int)((a.Lq + 15) / 16);
  const int64_t h = tile / qt, r0 = (int64_t)(tile % qt) * 16;
  const Walk<W> walk(a, r0);
  const int nb = walk.nb;
  const __amdgpu_buffer_rsrc_t rV = __builtin_amdgcn_make_buffer_rsrc((void*)(a.V + h * a.Lk * D + 16 * dt), (short)0,
                                                                    (int)(a.Lk * D * 2 - 32 * dt), 0x00020000);
  const __amdgpu_buffer_rsrc_t rP = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(s.ws + (int64_t)tile * s.nb_max * RF), (short)0, (int)((int64_t)nb * RF * 4), 0x00020000);
  // LDS row t of V (32 bytes) sits at t ^ 4 ((t / 8) % 2), so that the rows
  // 0..3 and 8..11 a transposing read's half wave takes lie on other banks
  auto vpos = [](int t) { return t ^ (((t >> 3) & 1) << 2); };
  const int vt = vpos(lane >> 1);               // the row this lane's 16 bytes belong to
  constexpr uint32_t OOB = 0x80000000u;
  uint32_t vof[NK], pof[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    vof[kk] = (uint32_t)((32 * kk + vt) * D * 2 + 16 * (lane & 1));
    pof[kk] = (uint32_t)(1024 * kk + 16 * lane);
  }
  const uint32_t aof = (uint32_t)((16 * W + 16 + li) * 4), rof = aof + 64;
  float al[RD], rs[RD];
  int sV = 0, sP = 0;                            // the next block's scalar offsets
  // loads of the next block (blocks are loaded in order), block b
  auto load = [&](char* slot, int u, int b) {
    const lds_char L = (lds_char)slot;
    int left = W;
    if constexpr (CAUSAL) {
      int kb = 0, ke = 0;
      if (b < nb) walk.block(b, &kb, &ke);
      sV = kb * D * 2;
      left = ke - kb;
    }
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const uint32_t off = !CAUSAL || 32 * kk + vt < left ? vof[kk] : OOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rV, (lds_void)(L + 1024 * kk), 16, off, sV, 0, 0);
    }
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const uint32_t off = pof[kk];
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rP, (lds_void)(L + 1024 * (NK + kk)), 16, off, sP, 0, 0);
    }
    al[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rP, aof, sP, 0));
    rs[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rP, rof, sP, 0));
    sV += W * D * 2;
    sP += RF * 4;
    __builtin_amdgcn_sched_barrier(0);
  };
  floatx4 O = {0.f, 0.f, 0.f, 0.f};
  float l = 0.f;
  const int vrow = 8 * G + (li >> 2), va = 32 * vpos(vrow) + 8 * (li & 3), vb = 32 * vpos(vrow + 4) + 8 * (li & 3);
  // fragments of the block being folded and of the next one, read from LDS a
  // block ahead
  shortx8 vf[2][NK], pf[2][NK];
  float ca[2], cr[2];
  auto read = [&](char* slot, int u, int x) {
    const lds_char L = (lds_char)slot;
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(L + 1024 * kk + va));
      const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(L + 1024 * kk + vb));
      vf[x][kk] = shortx8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
      pf[x][kk] = *(const shortx8*)(slot + 1024 * (NK + kk) + 16 * lane);
    }
    ca[x] = al[u];
    cr[x] = rs[u];
  };
  // block b in slot u, its fragments in set x: once they have arrived the slot
  // takes block b + RD, and block b + 1 (slot v) is read while b is folded
  auto step = [&](char* Lu, int u, char* Lv, int v, int x, int b) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_waitcnt(vmcnt_only((RD - 2) * PER));
    __builtin_amdgcn_sched_barrier(0);
    read(Lv, v, x ^ 1);
    load(Lu, u, b + RD);
    if (b < nb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) O[i] = ca[x] * O[i];
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) mfma_to(O, vf[x][kk], pf[x][kk]);
      l = a.l_fma ? __builtin_fmaf(ca[x], l, cr[x]) : ca[x] * l + cr[x];
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  static_for<0, RD>([&](auto u) { load(split_slot<W, u>(), u, u); });
  __builtin_amdgcn_s_waitcnt(vmcnt_only((RD - 1) * PER));
  __builtin_amdgcn_sched_barrier(0);
  read(split_slot<W, 0>(), 0, 0);
  for (int b = 0; b < nb; b += RD)
    static_for<0, RD>([&](auto u) {
      step(split_slot<W, u>(), u, split_slot<W, (u + 1) % RD>(), (u + 1) % RD, u % 2, b + u);
    });
  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));   // nothing lands in LDS after the wave has ended
  const int64_t row = r0 + li;
  if (row >= a.Lq) return;
  const float r = 1.0f / l;
  float y[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = a.final_recip ? O[e] * r : O[e] / l;
  const int64_t o = (h * a.Lq + row) * D + 16 * dt + 4 * G;
  if (a.out_bf16) *(uint2*)&((uint16_t*)a.O)[o] = uint2{f32x2_bf16x2(y[0], y[1]), f32x2_bf16x2(y[2], y[3])};
  else *(float4*)&((float*)a.O)[o] = float4{y[0], y[1], y[2], y[3]};
}

// ------------------------------------------------------------- launchers

static int64_t split_records(const AttnArgs& a, int W) {
  // a causal walk cuts at its query block's start: one block more at most
  return (a.Lk + W - 1) / W + (a.causal ? 1 : 0);
}

size_t attn_split_bytes(const AttnArgs& a, int key_block) {
  return (size_t)(a.H * ((a.Lq + 15) / 16)) * (size_t)split_records(a, key_block) * (16 * key_block + 48) * sizeof(float);
}

// When the split pays (speed only).  The one-launch kernels take about 20 us
// per 1000 keys (d = 128) however few the rows; the split three launches and,
// per tile, a pass over the records.  Measured on MI355X, one launch -> split,
// blocks of 64, d = 128:
//   tiles (heads x rows)      1024 keys       4096 keys
//   1    (1 x 1)              24.3 -> 15.0    84 -> 18
//   32   (32 x 1)             24.9 -> 14.7    85 -> 25
//   64   (64 x 16)            25.1 -> 15.8    86 -> 50
//   128  (32 x 64)            25.5 -> 22.8    86 -> 67
//   128  (128 x 16)           25.5 -> 23.9    88 -> 93    (K and V of 128 heads)
//   200  (200 x 1)            26.0 -> 37.0    92 -> 145
//   256  (1 x 4096, causal)                   85 -> 66
// so up to 64 tiles from 768 keys on (1024 for d = 64, whose one-launch blocks
// are shorter), beyond that only where the tiles share few heads' K and V.
bool attn_split_ok(const AttnArgs& a, int64_t dim, int key_block) {
  if (!a.block_tree || !a.pv_fma || a.Lk < (dim == 128 ? 768 : 1024) || a.H > 256 || a.Lq > 4096) return false;
  const int64_t tiles = a.H * ((a.Lq + 15) / 16);
  const bool fits = tiles <= 64 || (tiles <= 128 && (a.H <= 2 || (a.H <= 32 && a.Lk >= 2048))) ||
                    (tiles <= 256 && a.H <= 2 && a.Lk >= 2048);
  // V's rows and a tile's records within 31-bit offsets, with what attn_split_out
  // asks for past the end: its steps run to a whole ring and each loads a ring
  // further, 2 RD - 1 blocks (RD at most 8) and the offsets within a block
  return fits && (a.Lk + 16 * key_block) * dim * 2 <= 0x7fffffff &&
         (split_records(a, key_block) + 16) * (16 * key_block + 48) * 4 <= 0x7fffffff &&
         attn_split_bytes(a, key_block) <= (256u << 20);
}

template <int D, int W>
static hipError_t launch_split(const SplitArgs& s, hipStream_t st) {
  const dim3 grid((unsigned)((s.nb_max + 3) / 4), (unsigned)s.tiles), out((unsigned)((s.tiles + 7) / 8 * 8 * (D / 16)));
  hipLaunchKernelGGL((attn_split_scores<D, W>), grid, dim3(256), 0, st, s);
  hipLaunchKernelGGL((attn_split_probs<W>), grid, dim3(256), 0, st, s);
  constexpr int RD = W == 128 ? 6 : 8;
  if (s.a.causal) hipLaunchKernelGGL((attn_split_out<D, W, RD, true>), out, dim3(64), 0, st, s);
  else hipLaunchKernelGGL((attn_split_out<D, W, RD, false>), out, dim3(64), 0, st, s);
  return hipGetLastError();
}

hipError_t launch_attention_split(const AttnArgs& a, int64_t dim, int key_block, float* ws, hipStream_t st) {
  SplitArgs s;
  s.a = a;
  s.ws = ws;
  s.tiles = (int)(a.H * ((a.Lq + 15) / 16));
  s.nb_max = (int)split_records(a, key_block);
  if (dim == 64) {
    if (key_block == 32) return launch_split<64, 32>(s, st);
    if (key_block == 64) return launch_split<64, 64>(s, st);
    return launch_split<64, 128>(s, st);
  }
  if (key_block == 32) return launch_split<128, 32>(s, st);
  if (key_block == 64) return launch_split<128, 64>(s, st);
  return launch_split<128, 128>(s, st);
}

}  // namespace dg
