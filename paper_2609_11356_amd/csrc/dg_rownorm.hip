// dg_rownorm.hip -- row reductions and the normalisations on them (RMS norm,
// layer norm, softmax) with the row in registers, for the pinned leaf orders
// that dg_rowsum.hip defines: contiguous leaves of 64 (the count-up tree) and
// 64, 128 or 256 strided lanes.
//
// Bound: memory (X read once, Y written once).  A row is cut into passes of
// 4096 consecutive elements, one pass per wave (64 floats per lane), NW waves
// per row, so that a pass is an exact subtree (64 leaves of 64) or, over W
// strided lanes, 4096 / W consecutive steps of every lane's chain:
//   * contiguous leaves: each wave folds its 64 leaves through LDS (lane =
//     leaf, half a leaf at a time, 9 KB per wave), meets them by the count-up
//     butterfly, and the pass roots meet in the balanced tree;
//   * strided lanes: the waves fold in turn, each continuing the chains its
//     predecessor left in LDS; then the lanes meet.
// Missing elements hold -0, the exact identity of binary32 addition: s + -0
// keeps every s, and a square of -0 adds +0 to a sum of squares, which is
// never -0.  So no step needs a mask and the bits are those of the shorter
// sum.
//
// Rows of up to 65536 elements stay in registers from the load to the store
// (WIDE false); longer ones are walked in super-passes of 8 waves x 4096 by
// one workgroup and read again for every phase (WIDE true).  Loads and stores
// go in vectors whatever the row's alignment (4-byte aligned vector loads).
//
// Measured on MI355X (host-timed back to back, bf16 out) against the two to
// four passes through a workspace, which stay where they are the faster
// (row_fused_pays): layer norm 4096 x 4096
// 25.1 us (4.0 TB/s) from 82.8, 64 x 32768 12.3 from 107; softmax 4096 x 16384
// 93 us (4.3 TB/s) from 314, 64 x 100000 26 from 322; RMS norm 16384 x 4096
// 100 us from 127; row sums of 64 x 32768 7.7 us from 18.6.
#include <type_traits>

#include "dg_rows.h"

namespace dg {

namespace {

constexpr int PASS = 4096;           // elements of a row per wave
constexpr int LEAF_PITCH = 36;       // floats between leaves in LDS (32 + 4: 16-byte rows, spread over the banks)
constexpr int MAX_PASSES = 2048;     // pass roots of a WIDE row in LDS (rows of up to 8.4 M elements)

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
// the same with element alignment: one vector access wherever the row starts
typedef f4 f4u __attribute__((aligned(4)));
typedef f2 f2u __attribute__((aligned(4)));
typedef uint16_t h4 __attribute__((ext_vector_type(4)));
typedef uint16_t h2 __attribute__((ext_vector_type(2)));
typedef h4 h4u __attribute__((aligned(2)));
typedef h2 h2u __attribute__((aligned(2)));

template <int V>
__device__ __forceinline__ void load_f32(const float* p, float* v) {
  if constexpr (V == 4) {
    const f4 f = *(const f4u*)p;
    v[0] = f[0]; v[1] = f[1]; v[2] = f[2]; v[3] = f[3];
  } else if constexpr (V == 2) {
    const f2 f = *(const f2u*)p;
    v[0] = f[0]; v[1] = f[1];
  } else {
    v[0] = *p;
  }
}

template <int V>
__device__ __forceinline__ void load_bf16(const uint16_t* p, float* v) {
  if constexpr (V == 4) {
    const h4 h = *(const h4u*)p;
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = bf16_f32(h[u]);
  } else if constexpr (V == 2) {
    const h2 h = *(const h2u*)p;
    v[0] = bf16_f32(h[0]); v[1] = bf16_f32(h[1]);
  } else {
    v[0] = bf16_f32(*p);
  }
}

template <int V>
__device__ __forceinline__ void store_f32(float* p, const float* y) {
  if constexpr (V == 4) *(f4u*)p = f4{y[0], y[1], y[2], y[3]};
  else if constexpr (V == 2) *(f2u*)p = f2{y[0], y[1]};
  else *p = y[0];
}

template <int V>
__device__ __forceinline__ void store_bf16(uint16_t* p, const float* y) {
  if constexpr (V == 4) {
    const uint32_t lo = f32x2_bf16x2(y[0], y[1]), hi = f32x2_bf16x2(y[2], y[3]);
    *(h4u*)p = h4{(uint16_t)lo, (uint16_t)(lo >> 16), (uint16_t)hi, (uint16_t)(hi >> 16)};
  } else if constexpr (V == 2) {
    const uint32_t lo = f32x2_bf16x2(y[0], y[1]);
    *(h2u*)p = h2{(uint16_t)lo, (uint16_t)(lo >> 16)};
  } else {
    *p = f32_bf16(y[0]);
  }
}

// Consecutive elements a lane holds per slot, and a slot's first element
// within the wave's pass.  W = 0: contiguous leaves (slot t = 8 h + j covers
// half h of leaves 8 j .. 8 j + 7, eight lanes a leaf: 128-byte runs).
template <int W>
constexpr int row_vec() { return W == 0 || W == 256 ? 4 : W == 128 ? 2 : 1; }
template <int W>
__device__ __forceinline__ int slot_off(int t, int lane) {
  if constexpr (W == 0) return (8 * (t & 7) + (lane >> 3)) * 64 + 32 * (t >> 3) + 4 * (lane & 7);
  else return t * W + lane * row_vec<W>();
}

// The pass at p (element `base` of the row), elements at or past cols as pad.
template <int W>
__device__ __forceinline__ void load_pass(float (&v)[64], const float* x, int64_t base, int64_t cols, int lane,
                                          float pad) {
  constexpr int V = row_vec<W>();
  const float* p = x + base;
  if (base + PASS <= cols) {
#pragma unroll
    for (int t = 0; t < 64 / V; ++t) load_f32<V>(p + slot_off<W>(t, lane), &v[V * t]);
  } else {
    const int n = (int)(cols - base);
#pragma unroll
    for (int t = 0; t < 64 / V; ++t) {
      const int e = slot_off<W>(t, lane);
      if (e + V <= n) {
        load_f32<V>(p + e, &v[V * t]);
      } else {
#pragma unroll
        for (int u = 0; u < V; ++u) v[V * t + u] = e + u < n ? p[e + u] : pad;
      }
    }
  }
}

// -0 in every missing element of a pass (after a step that changed them).
template <int W>
__device__ __forceinline__ void repad(float (&v)[64], int64_t base, int64_t cols, int lane) {
  constexpr int V = row_vec<W>();
  if (base + PASS <= cols) return;
  const int n = (int)(cols - base);
#pragma unroll
  for (int t = 0; t < 64 / V; ++t)
#pragma unroll
    for (int u = 0; u < V; ++u) v[V * t + u] = slot_off<W>(t, lane) + u < n ? v[V * t + u] : -0.0f;
}

// Compiler and wave order of LDS phases (a wave's LDS operations run in issue order).
__device__ __forceinline__ void lds_phase() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// OP: 0 sum, 1 sum of squares by fused square-add, 2 by a rounded square.
template <int OP>
__device__ __forceinline__ float fold_step(float s, float x) { return leaf_step(s, x, OP > 0, OP == 1); }

// A pass of contiguous leaves: every lane folds leaf `lane` in index order
// (starting at -0, which the first element replaces exactly), then the
// count-up butterfly.  sl: the wave's 64 x LEAF_PITCH floats.
template <int OP>
__device__ __forceinline__ float pass_root(const float (&v)[64], float* sl, int lane) {
  float s = -0.0f;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    lds_phase();
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int t = 8 * h + j;
      *(f4*)&sl[(8 * j + (lane >> 3)) * LEAF_PITCH + 4 * (lane & 7)] = f4{v[4 * t], v[4 * t + 1], v[4 * t + 2], v[4 * t + 3]};
    }
    lds_phase();
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const f4 x = *(const f4*)&sl[lane * LEAF_PITCH + 4 * q];
#pragma unroll
      for (int u = 0; u < 4; ++u) s = fold_step<OP>(s, x[u]);
    }
  }
  return tree_sum_lanes<6>(s);
}

__device__ __forceinline__ float wave_max(float m) { return max_lanes<6>(m); }

// The maximum of a pass.  A NaN is ignored here: its own exponential is NaN,
// which makes the row's sum, its reciprocal and every output NaN, as a NaN
// maximum would.
__device__ __forceinline__ float pass_max(const float (&v)[64]) {
  float m = -__builtin_inff();
#pragma unroll
  for (int i = 0; i < 64; ++i) m = __builtin_fmaxf(m, v[i]);
  return m;
}

// Scale a pass and store it: y = v rinv, optionally rounded to bf16, times w,
// plus b.
template <int W, bool NORM>
__device__ __forceinline__ void store_pass(const float (&v)[64], const NormArgs& a, float rinv, int64_t row,
                                           int64_t base, int lane) {
  constexpr int V = row_vec<W>();
  const int64_t left = a.cols - base;
  const int n = left < PASS ? (int)left : PASS;
  const uint16_t* w = NORM && a.w ? a.w + base : nullptr;
  const uint16_t* b = NORM && a.b ? a.b + base : nullptr;
  const int64_t o = row * a.cols + base;
  auto finish = [&](float x, bool hw, float wv, bool hb, float bv) {
    float y = x * rinv;
    if constexpr (NORM) {
      if (a.pre_round) y = round_bf16(y);
      if (hw) y = y * wv;
      if (hb) y = y + bv;
    }
    return y;
  };
#pragma unroll
  for (int t = 0; t < 64 / V; ++t) {
    const int e = slot_off<W>(t, lane);
    if (e + V <= n) {
      float wv[V], bv[V], y[V];
      if (w) load_bf16<V>(w + e, wv);
      if (b) load_bf16<V>(b + e, bv);
#pragma unroll
      for (int u = 0; u < V; ++u) y[u] = finish(v[V * t + u], w != nullptr, wv[u], b != nullptr, bv[u]);
      if (a.out_bf16) store_bf16<V>((uint16_t*)a.Y + o + e, y);
      else store_f32<V>((float*)a.Y + o + e, y);
    } else {
#pragma unroll
      for (int u = 0; u < V; ++u)
        if (e + u < n) {
          const float y = finish(v[V * t + u], w != nullptr, w ? bf16_f32(w[e + u]) : 0.f, b != nullptr,
                                 b ? bf16_f32(b[e + u]) : 0.f);
          if (a.out_bf16) ((uint16_t*)a.Y)[o + e + u] = f32_bf16(y);
          else ((float*)a.Y)[o + e + u] = y;
        }
    }
  }
}

}  // namespace

// KIND: ROW_*.  W: strided lanes, or 0 for contiguous leaves of 64.  SQ: the
// sum (ROW_SUM) is one of squares.  Squares join by one fused square-add (a
// descriptor with fma = 0 takes the passes of dg_rowsum.hip).  NW waves per
// row, max(4, NW) per workgroup.  A WIDE row runs on eight waves: its walk
// needs more than the 128 registers per lane that sixteen would leave.
template <int KIND, int W, bool SQ, int NW, bool WIDE>
__global__ __launch_bounds__(64 * (NW < 4 ? 4 : NW)) __attribute__((amdgpu_waves_per_eu(WIDE ? 2 : 4))) void row_fused(
    RowsumArgs ra, NormArgs a) {
  static_assert(!WIDE || NW == 8, "wide rows take a whole workgroup");
  constexpr int NWG = NW < 4 ? 4 : NW, RPG = NWG / NW, V = row_vec<W>();
  constexpr int NROOT = WIDE ? MAX_PASSES : NWG;
  __shared__ __attribute__((aligned(16))) float stage[W == 0 ? NWG * 64 * LEAF_PITCH : 4];
  __shared__ float roots[W == 0 ? 2 : 1][W == 0 ? NROOT : 1];
  __shared__ __attribute__((aligned(16))) float hand[W == 0 ? 1 : 2][W == 0 ? 1 : RPG * W];
  __shared__ float wmax[KIND == ROW_SMX ? NWG : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int rg = wave / NW, wr = wave % NW;   // the row within the workgroup, the wave within the row
  const int64_t row = (int64_t)blockIdx.x * RPG + rg;
  const bool live = row < a.rows;
  const int64_t cols = a.cols;
  const float* x = a.X + (live ? row : 0) * cols;
  const int64_t nsp = WIDE ? (cols + (int64_t)PASS * NW - 1) / ((int64_t)PASS * NW) : 1;
  auto base_of = [&](int64_t sp) { return (sp * NW + wr) * (int64_t)PASS; };
  constexpr bool SMX = KIND == ROW_SMX;
  float v[64];

  // the row's sum over f(pass) (f leaves the pass in v, -0 where missing);
  // `which` names the LDS area, so that two sums of a row need no barrier between
  auto total = [&](auto op_, int which, auto f) -> float {
    constexpr int O = decltype(op_)::value;
    if constexpr (W == 0) {
      float r = -0.0f;
      for (int64_t sp = 0; sp < nsp; ++sp) {
        const int64_t base = base_of(sp);
        r = -0.0f;
        if (base < cols) {
          f(base);
          r = pass_root<O>(v, &stage[wave * 64 * LEAF_PITCH], lane);
        }
        if (NW > 1 && lane == 0) roots[which][WIDE ? sp * NW + wr : wave] = r;
      }
      if constexpr (NW == 1) return r;
      __syncthreads();
      if constexpr (!WIDE) {
        float t[NW];
#pragma unroll
        for (int g = 0; g < NW; ++g) t[g] = roots[which][rg * NW + g];
#pragma unroll
        for (int h = 1; h < NW; h <<= 1)
#pragma unroll
          for (int g = 0; g < NW; g += 2 * h) t[g] = t[g] + t[g + h];
        return t[0];
      } else {
        // the balanced tree over the nsp NW roots, level by level; a missing
        // partner is -0
        float* R = roots[which];
        const int np = (int)(nsp * NW);
        for (int h = 1; h < np; h <<= 1) {
          for (int i = 2 * h * (int)threadIdx.x; i < np; i += 2 * h * 64 * NWG)
            if (i + h < np) R[i] = R[i] + R[i + h];
          __syncthreads();
        }
        return R[0];
      }
    } else {
      float s[V];
#pragma unroll
      for (int u = 0; u < V; ++u) s[u] = -0.0f;
      float* hb = &hand[which][rg * W + lane * V];
      for (int64_t sp = 0; sp < nsp; ++sp) {
        const int64_t base = base_of(sp);
        if (base < cols) f(base);
#pragma unroll 1
        for (int g = 0; g < NW; ++g) {
          if (wr == g && base < cols) {
            if (g > 0 || sp > 0) {
#pragma unroll
              for (int u = 0; u < V; ++u) s[u] = hb[u];
            }
#pragma unroll
            for (int t = 0; t < 64 / V; ++t)
#pragma unroll
              for (int u = 0; u < V; ++u) s[u] = fold_step<O>(s[u], v[V * t + u]);
            if constexpr (NW > 1) {
#pragma unroll
              for (int u = 0; u < V; ++u) hb[u] = s[u];
            }
          }
          if constexpr (NW > 1) __syncthreads();
        }
      }
      if constexpr (NW > 1) {
#pragma unroll
        for (int u = 0; u < V; ++u) s[u] = hb[u];
      }
      return ra.down ? lanes_meet<V, true>(s) : lanes_meet<V, false>(s);
    }
  };
  using op_sum = std::integral_constant<int, 0>;
  using op_own = std::integral_constant<int, KIND == ROW_SUM ? (SQ ? 1 : 0) : 1>;

  if constexpr (!WIDE) {
    if (base_of(0) < cols) load_pass<W>(v, x, base_of(0), cols, lane, SMX ? -__builtin_inff() : -0.0f);
  }
  auto get = [&](int64_t base) {
    if constexpr (WIDE) load_pass<W>(v, x, base, cols, lane, SMX ? -__builtin_inff() : -0.0f);
  };

  float m = 0.f, mean = 0.f, rinv = 0.f;
  if constexpr (KIND == ROW_SUM || KIND == ROW_RMS) {
    const float s = total(op_own{}, 0, [&](int64_t base) { get(base); });
    if constexpr (KIND == ROW_SUM) {
      if (live && wr == 0 && lane == 0) ra.out[row] = s;
      return;
    }
    rinv = rms_inv(s, cols, ra.eps);
  } else if constexpr (KIND == ROW_LN) {
    mean = total(op_sum{}, 0, [&](int64_t base) { get(base); }) / (float)cols;
    rinv = rms_inv(total(op_own{}, 1,
                         [&](int64_t base) {
                           get(base);
#pragma unroll
                           for (int i = 0; i < 64; ++i) v[i] = v[i] - mean;
                           repad<W>(v, base, cols, lane);
                         }),
                   cols, ra.eps);
  } else {
    m = -__builtin_inff();
    for (int64_t sp = 0; sp < nsp; ++sp)
      if (base_of(sp) < cols) {
        get(base_of(sp));
        m = __builtin_fmaxf(m, pass_max(v));
      }
    m = wave_max(m);
    if constexpr (NW > 1) {
      if (lane == 0) wmax[wave] = m;
      __syncthreads();
#pragma unroll
      for (int g = 0; g < NW; ++g) m = __builtin_fmaxf(m, wmax[rg * NW + g]);
    }
    rinv = 1.0f / total(op_sum{}, 0, [&](int64_t base) {
             get(base);
#pragma unroll
             for (int i = 0; i < 64; ++i) v[i] = exp_nonpos(v[i] - m);
             repad<W>(v, base, cols, lane);
           });
  }

  if constexpr (KIND != ROW_SUM) {
    if (!live) return;
    for (int64_t sp = 0; sp < nsp; ++sp) {
      const int64_t base = base_of(sp);
      if (base >= cols) continue;
      if constexpr (WIDE) {
        get(base);
        if constexpr (KIND == ROW_LN) {
#pragma unroll
          for (int i = 0; i < 64; ++i) v[i] = v[i] - mean;
        } else if constexpr (KIND == ROW_SMX) {
#pragma unroll
          for (int i = 0; i < 64; ++i) v[i] = exp_nonpos(v[i] - m);
        }
      }
      store_pass<W, KIND != ROW_SMX>(v, a, rinv, row, base, lane);
    }
  }
}

// ------------------------------------------------------------- launchers

// Waves per row: the power of two that gives every wave at most one pass
// (strided lanes, whose short aligned rows have their own kernels, are built
// for 1, 4 and 16 only).
template <int KIND, int W, bool SQ>
static hipError_t launch_rf(const RowsumArgs& r, const NormArgs& a, hipStream_t st) {
  const int64_t np = (a.cols + PASS - 1) / PASS;
  auto go = [&](auto nw_, auto wide_) {
    constexpr int NW = decltype(nw_)::value, NWG = NW < 4 ? 4 : NW, RPG = NWG / NW;
    hipLaunchKernelGGL((row_fused<KIND, W, SQ, NW, decltype(wide_)::value>),
                       dim3((unsigned)((a.rows + RPG - 1) / RPG)), dim3(64 * NWG), 0, st, r, a);
  };
  using std::integral_constant;
  if (np > 16) go(integral_constant<int, 8>{}, std::true_type{});
  else if constexpr (W == 0) {
    if (np <= 1) go(integral_constant<int, 1>{}, std::false_type{});
    else if (np <= 2) go(integral_constant<int, 2>{}, std::false_type{});
    else if (np <= 4) go(integral_constant<int, 4>{}, std::false_type{});
    else if (np <= 8) go(integral_constant<int, 8>{}, std::false_type{});
    else go(integral_constant<int, 16>{}, std::false_type{});
  } else {
    if (np <= 1) go(integral_constant<int, 1>{}, std::false_type{});
    else if (np <= 4) go(integral_constant<int, 4>{}, std::false_type{});
    else go(integral_constant<int, 16>{}, std::false_type{});
  }
  return hipGetLastError();
}

template <int W>
hipError_t launch_row_fused_w(const RowsumArgs& r, const NormArgs& a, int kind, hipStream_t st) {
  switch (kind) {
    case ROW_SUM: return r.sumsq ? launch_rf<ROW_SUM, W, true>(r, a, st) : launch_rf<ROW_SUM, W, false>(r, a, st);
    case ROW_RMS: return launch_rf<ROW_RMS, W, false>(r, a, st);
    case ROW_LN: return launch_rf<ROW_LN, W, false>(r, a, st);
    case ROW_SMX: return launch_rf<ROW_SMX, W, false>(r, a, st);
  }
  return hipErrorInvalidValue;
}

#ifdef DG_ROWNORM_STRIDED
template hipError_t launch_row_fused_w<64>(const RowsumArgs&, const NormArgs&, int, hipStream_t);
template hipError_t launch_row_fused_w<128>(const RowsumArgs&, const NormArgs&, int, hipStream_t);
template hipError_t launch_row_fused_w<256>(const RowsumArgs&, const NormArgs&, int, hipStream_t);
#else
extern template hipError_t launch_row_fused_w<64>(const RowsumArgs&, const NormArgs&, int, hipStream_t);
extern template hipError_t launch_row_fused_w<128>(const RowsumArgs&, const NormArgs&, int, hipStream_t);
extern template hipError_t launch_row_fused_w<256>(const RowsumArgs&, const NormArgs&, int, hipStream_t);

// Whether a call can run here: contiguous leaves of 64 or 64, 128, 256 strided
// lanes, any alignment and length up to the pass roots LDS holds; squares by
// the fused square-add.
bool row_fused_can(const RowsumArgs& r, int kind, int64_t cols) {
  if (cols < 1 || cols > (int64_t)MAX_PASSES * PASS) return false;
  if ((kind == ROW_RMS || kind == ROW_LN || r.sumsq) && !r.fma) return false;
  return r.strided ? (r.leaf_w == 64 || r.leaf_w == 128 || r.leaf_w == 256) : r.leaf_w == 64;
}

// Whether one that can should (speed only: the kernels of dg_rowsum.hip, one
// wave per row in one to four launches, give the same bits).
//
// The lines below are where the two cross on MI355X (operands from HBM, bf16
// out, us, one wave a row -> here).  A row of np passes holds the 1, 4 or 16
// waves it is built for whatever np is, and over strided lanes the waves fold
// in turn, so the cost here is per row and round of the chip (256 rows of 5 to
// 16 passes, or of more); there it is per element, and several times higher
// where a row starts off the vector loads (`al` false).
bool row_fused_pays(const RowsumArgs& r, int kind, int64_t rows, int64_t cols, int ncu) {
  const int64_t np = (cols + PASS - 1) / PASS, rounds = (rows + ncu - 1) / ncu;
  const bool al = cols % 4 == 0 && ((uintptr_t)r.X & 15) == 0, full = cols % PASS == 0;
  const int W = r.strided ? r.leaf_w : 0;
  // Rows past 65536 elements are read again for each phase: once there are rows
  // enough for the other path to fill the chip as well, an RMS norm (one read
  // more either way) and a layer norm over 64 lanes stay there (1000 x 131072:
  // 277 against 299, 871 against 927).
  if (np > 16 && rows >= 512 && (kind == ROW_RMS || (kind == ROW_LN && W == 64))) return false;
  if (W == 0) {
    // an RMS norm of aligned short rows is two short launches there: 1000 x 640
    // 7.5 -> 8.0, 2000 x 768 8.3 -> 9.5, 64 x 3000 7.4 -> 8.4; fewer rows or
    // more, 1 x 640 7.0 -> 6.3, 4096 x 1000 14.5 -> 12.7, 2000 x 3000 15.1 -> 13.8
    return !(kind == ROW_RMS && al && cols < PASS &&
             ((cols <= 1024 && rows > ncu && rows <= 8 * ncu) || (cols > 2048 && rows > 4 && rows <= 2 * ncu)));
  }
  if (np == 1) {
    // (unaligned: aligned rows have their own kernels)  a wave here walks all 64
    // slots however short the row: 16384 x 65 over 128 lanes RMS norm 11.4 ->
    // 25.5, softmax 25 -> 38, layer norm 23 -> 31; 1000 x 65 7.0 -> 6.4, 9.6 -> 7.4,
    // 12.5 -> 7.8.  Over 64 lanes both take as long.
    if (W == 64) return true;
    if (kind == ROW_RMS) return !(cols < 768 && rows > (cols < 512 ? 8 : 16) * (int64_t)ncu);
    if (kind == ROW_LN) return !(cols < 192 && rows > 16 * (int64_t)ncu);
    if (kind == ROW_SMX) return !(cols < 256 && rows > 8 * (int64_t)ncu);
    return true;
  }
  if (kind == ROW_SMX) return true;   // three launches there
  // layer norm: over 64 lanes the longest turns: 1500 x 24576 193 -> 247, 768 x 24576 118 -> 119
  if (kind == ROW_LN) return !(W == 64 && np >= 5 && np <= 8 && rounds > 3 && !(np == 5 && !al));
  if (kind == ROW_SUM) {
    // one launch either way.  256 lanes: 256 x 32769 17 -> 12, 400 x 32769 20 ->
    // 22, 768 x 32769 26 -> 39, 400 x 65536 33 -> 28; 64 lanes: 768 x 32768 33 -> 23,
    // 1000 x 40000 37 -> 50
    if (np <= 4) return true;
    if (rounds <= 1) return rows > 1 || np > 5;
    if (rounds == 2) return W < 256 || full || np >= 10;
    if (rounds == 3 && W == 64 && np > 5) return true;
    return W < 256 && full;
  }
  // RMS norm: two launches there.  64 lanes: 128 x 32768 40 -> 30, 512 x 32768
  // 53 -> 64, 1000 x 20000 42 -> 99, 500 x 32769 93 -> 63, 1000 x 8196 25 -> 31,
  // 6000 x 8196 102 -> 93; 128 lanes: 256 x 20000 27 -> 19, 1000 x 20000 42 ->
  // 65, 1000 x 32769 113 -> 96, 2000 x 16385 89 -> 101, 4175 x 16499 224 -> 207;
  // 256 lanes: 500 x 20000 29 -> 26, 1000 x 20000 41 -> 49, 1000 x 32768 65 ->
  // 62
  if (np > 16) {
    if (!al) return true;
    return W == 64 ? rows <= 32 : rounds <= 1 || (W == 256 && np >= 21);
  }
  if (np <= 4) {
    if (W == 64) return !al || (full ? rows > 1 && rounds <= 4 : rounds > 20);
    return !(al && W == 128 && rows < 4);
  }
  if (!al) return W == 64 ? rounds <= (np <= 8 ? 2 : 3) : W == 128 ? rounds <= 3 || np > 8 || (np == 5 && rounds > 10) : true;
  if (W == 64) return (rounds <= 1 && (rows > 1 || np > 5)) || (rounds == 2 && np >= 12);
  if (W == 128) return rounds <= 1 || (rounds == 2 && (full || np > 8)) || np >= 12;
  return rounds <= 2 || np >= 8;
}

hipError_t launch_row_fused(const RowsumArgs& r, const NormArgs& a, int kind, hipStream_t st) {
  if (!r.strided) return launch_row_fused_w<0>(r, a, kind, st);
  switch (r.leaf_w) {
    case 64: return launch_row_fused_w<64>(r, a, kind, st);
    case 128: return launch_row_fused_w<128>(r, a, kind, st);
    case 256: return launch_row_fused_w<256>(r, a, kind, st);
  }
  return hipErrorInvalidValue;
}

// Softmax of few wide rows (contiguous leaves): every pass of every row on a
// wave of its own, in three launches, because one workgroup per row leaves
// most of the chip idle and the exponentials of a 100000-element row alone
// take a CU 15 us.  PHASE 0: the pass maxima (part).  PHASE 1: the pass roots
// of the exponentials (root).  PHASE 2: the roots meet (npass <= 64, one per
// lane), and the outputs.  X is read three times (from the caches after the
// first) and its exponentials computed twice, which costs less than writing
// them out and reading them back.
template <int PHASE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void softmax_split(NormArgs a, float* part,
                                                                                             float* root, int npass) {
  __shared__ __attribute__((aligned(16))) float stage[PHASE == 1 ? 4 * 64 * LEAF_PITCH : 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t unit = (int64_t)blockIdx.x * 4 + wave;   // (row, pass)
  const int64_t row = unit / npass;
  const int p = (int)(unit % npass);
  if (row >= a.rows) return;   // whole waves; no barrier below
  const int64_t base = (int64_t)p * PASS;
  float v[64];
  load_pass<0>(v, a.X + row * a.cols, base, a.cols, lane, -__builtin_inff());
  if constexpr (PHASE == 0) {
    const float m = wave_max(pass_max(v));
    if (lane == 0) part[row * npass + p] = m;
  } else {
    const float m = wave_max(lane < npass ? part[row * npass + lane] : -__builtin_inff());
#pragma unroll
    for (int i = 0; i < 64; ++i) v[i] = exp_nonpos(v[i] - m);
    if constexpr (PHASE == 1) {
      repad<0>(v, base, a.cols, lane);
      const float r = pass_root<0>(v, &stage[wave * 64 * LEAF_PITCH], lane);
      if (lane == 0) root[row * npass + p] = r;
    } else {
      const float s = tree_sum_lanes<6>(lane < npass ? root[row * npass + lane] : -0.0f);
      store_pass<0, false>(v, a, 1.0f / s, row, base, lane);
    }
  }
}

bool softmax_split_ok(const RowsumArgs& r, int64_t rows, int64_t cols) {
  return !r.strided && r.leaf_w == 64 && cols > 16 * PASS && cols <= 64 * PASS && rows < 256;
}

size_t softmax_split_bytes(int64_t rows, int64_t cols) {
  return (size_t)rows * (size_t)((cols + PASS - 1) / PASS) * 2 * sizeof(float);
}

hipError_t launch_softmax_split(const NormArgs& a, float* ws, hipStream_t st) {
  const int npass = (int)((a.cols + PASS - 1) / PASS);
  const int64_t units = a.rows * npass;
  float* root = ws + units;
  const dim3 grid((unsigned)((units + 3) / 4)), block(256);
  hipLaunchKernelGGL((softmax_split<0>), grid, block, 0, st, a, ws, root, npass);
  hipLaunchKernelGGL((softmax_split<1>), grid, block, 0, st, a, ws, root, npass);
  hipLaunchKernelGGL((softmax_split<2>), grid, block, 0, st, a, ws, root, npass);
  return hipGetLastError();
}
#endif

}  // namespace dg
