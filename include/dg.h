/*
 * dg.h -- descriptor-ordered bf16 GEMM and row reduction for MI355X (gfx950).
 *
 * C ABI of libdg.so.  Every floating-point reduction order the library
 * computes is fixed by a descriptor, never by the tile shape, wave count or
 * grid the library picks for speed, so the bits of every output depend only
 * on the descriptor and the operands -- not on M, on other rows, or on the
 * launch configuration.
 *
 * Paper: "Taming Bitwise Behavior in GPU Kernels with Tensor Core" --
 *   Sec. 3.1  a reduction's order is its dependence tree; equal trees (up to
 *             swapping children) give equal bits;
 *   Sec. 3.2.1 a matrix instruction folds a group of products and the
 *             accumulator with its own rounding rule;
 *   Sec. 3.2.2 the GEMM descriptor: instruction_k, use_fast_accum,
 *             k_loop_step, split-K span / k_cuts, partial_dtype, merge_dtype;
 *   Sec. 5.1  the balanced (count-up) tree used for every tree combine.
 *
 * Conventions (all entry points):
 *   - No exception crosses the ABI; every entry point returns a dg_status.
 *   - Device pointers are caller-owned HIP device allocations; the library
 *     never frees them.  Matrices are dense row-major: A is M x K (leading
 *     dimension K), B is K x N (N), C is M x N (N), X is rows x cols (cols).
 *     bf16 operands are raw IEEE bfloat16 bit patterns (uint16).
 *   - `stream` is a hipStream_t (NULL = the default stream).  Work is enqueued
 *     and the call returns; results are ready when the stream reaches them.
 *   - Validation happens before anything is enqueued: an error return means
 *     nothing was launched and no output was written.
 *   - A descriptor is immutable after dg_desc_create and may be used from any
 *     number of host threads and streams at once.
 *   - Library-owned workspaces are kept per (device, stream handle), grow in
 *     stream order and stay until the process ends.  Under hipStreamPerThread,
 *     one handle for a stream of every host thread, a call allocates and frees
 *     its own in stream order instead.  A stream may be destroyed only when its
 *     work is done, as a later stream can get the same handle.  A captured call
 *     keeps the workspace it found, so a call of its size must have run on the
 *     stream before, and the graph must not be replayed after one that needs
 *     more (dg_gemm_noalloc, and calls that take no workspace, never do).
 */
#ifndef DG_H
#define DG_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

typedef enum {
  DG_OK = 0,
  DG_ERR_INVALID = 1,     /* a NULL handle/pointer or a field out of range */
  DG_ERR_UNSUPPORTED = 2, /* a valid order this build cannot realise */
  DG_ERR_SHAPE = 3,       /* sizes inconsistent with the descriptor's plan */
  DG_ERR_ALIGN = 4,       /* a device pointer not aligned to its element size */
  DG_ERR_NOMEM = 5,       /* split-K workspace allocation failed */
  DG_ERR_HIP = 6,         /* a HIP runtime call or kernel launch failed */
  DG_ERR_SCRATCH = 7      /* dg_gemm_noalloc: S * M * N partials exceed its
                             fixed scratch (DG_NOALLOC_SCRATCH_BYTES) */
} dg_status;

/* Matrix instruction whose group the descriptor names (Sec. 3.2.1:
 * instruction_k).  On gfx950 both bf16 instructions fold their products in
 * chunks of 8 consecutive k; with fma = 1 they therefore give the same bits,
 * and with fma = 0 the instruction's K (32 or 16) is the group rounded on its
 * own before it meets the accumulator. */
enum { DG_MMA_16X16X32_BF16 = 1, /* group of 32 */
       DG_MMA_32X32X16_BF16 = 2, /* group of 16 */
       DG_MMA_SCALAR_FMA = 3,    /* group of 1: each product joins the accumulator
                                    by one binary32 fused multiply-add (the scalar
                                    path of chained chunks, Sec. 3.2.2); fma has no
                                    effect (a bf16 product is exact); any tile_k */
       /* The fp8 instructions (in_dtype DG_IN_E4M3 only; Sec. 3.2.1: their
        * semantics are their own).  On gfx950 all four fold their products
        * in chunks of 16 consecutive k, each two groups of 8 truncated onto
        * 2^(E_g - 13), the group sums floored onto 2^(E - 24), an
        * accumulator below 2^(E - 25) left out, one rounding per chunk; so
        * with fma = 1 they give the same bits, and with fma = 0 the
        * instruction's K is the group.  The block-scaled f8f6f4 shapes are
        * taken with e4m3 operands and unit scales. */
       DG_MMA_16X16X32_FP8 = 4,     /* group of 32 */
       DG_MMA_32X32X16_FP8 = 5,     /* group of 16 */
       DG_MMA_16X16X128_F8F6F4 = 6, /* group of 128 */
       DG_MMA_32X32X64_F8F6F4 = 7   /* group of 64 */ };
enum { DG_CARRY = 0, DG_SEQ = 1, DG_TREE = 2 };  /* combine rules */
enum { DG_TAIL_LAST = 0, DG_TAIL_FIRST = 1 };     /* short K tile position (k_loop_step) */
enum { DG_F32 = 0, DG_BF16 = 1 };                  /* storage/rounding types */
enum { DG_EPI_NONE = 0, DG_EPI_BIAS = 1, DG_EPI_BIAS_SILU = 2 };
enum { DG_ROUND_FINAL = 0, DG_ROUND_PRE_ACT = 1 };
enum { DG_OP_SUM = 0, DG_OP_SUMSQ = 1 };
enum { DG_SPLIT_CONTIGUOUS = 0, DG_SPLIT_STRIDED = 1 };  /* layout of the split (Sec. 3.2.2) */
enum { DG_LEAF_CONTIGUOUS = 0, DG_LEAF_STRIDED = 1 };    /* row-reduction leaf layout */
enum { DG_FOLD_UP = 0, DG_FOLD_DOWN = 1 };               /* how the leaves meet */
enum { DG_NORM_FINAL = 0, DG_NORM_PRE_WEIGHT = 1 };      /* RMS-norm rounding point */
enum { DG_IN_BF16 = 0, DG_IN_F16 = 1, DG_IN_BF16_E4M3 = 2, DG_IN_E4M3 = 3 }; /* GEMM operand format */

#define DG_MAX_SPLIT 64
#define DG_SIGNATURE_MAX 2048
#define DG_NOALLOC_SCRATCH_BYTES (16u << 20) /* dg_gemm_noalloc's fixed split-K scratch */

/* The order fields, and nothing else (Sec. 3.2.2; Sec. 4 keeps a reconstructed
 * order as a frozen record of all of its factors).  No speed knob appears here. */
typedef struct {
  uint32_t struct_size;   /* sizeof(dg_desc_params), for ABI versioning */
  int32_t mma;            /* DG_MMA_*: the instruction group */
  int32_t tile_k;         /* K tile: an accumulator may close every tile_k
                             elements of a part; a multiple of the group */
  int32_t split_k;        /* number of K parts S, 1..DG_MAX_SPLIT (Sec. 3.2.2 split-K) */
  int32_t n_cuts;         /* 0: span rule; else S-1 explicit interior cuts */
  const int64_t* k_cuts;  /* host array of n_cuts strictly increasing cut
                             points in (0, K); copied at create time */
  int32_t tile_combine;   /* DG_CARRY: one accumulator through the part;
                             DG_SEQ / DG_TREE: each tile from +0, tiles
                             chained / combined by the balanced tree */
  int32_t split_combine;  /* DG_SEQ or DG_TREE over the S parts (second kernel) */
  int32_t tail;           /* DG_TAIL_LAST / DG_TAIL_FIRST: where a part's short
                             tile sits (k_loop_step) */
  int32_t fma;            /* 1: the accumulator is the instruction's C operand
                             (use_fast_accum off: one rounding per step);
                             0: each group from +0, then a separate add */
  int32_t partial_dtype;  /* DG_F32 / DG_BF16: type a finished part is written at */
  int32_t merge_dtype;    /* DG_F32 / DG_BF16: type of the running merge sum
                             (DG_BF16 requires partial_dtype DG_BF16) */
  int32_t out_dtype;      /* DG_F32 / DG_BF16: C element type */
  int32_t epilogue;       /* DG_EPI_*: z = y (+) bias_j, then SiLU */
  int32_t epi_round;      /* DG_ROUND_FINAL: out = RN_out(silu(z));
                             DG_ROUND_PRE_ACT: out = RN_bf16(silu(RN_bf16(z)))
                             (requires DG_EPI_BIAS_SILU) */
  int32_t leaf_w;         /* row reduction: elements folded in index order per
                             leaf before the balanced tree over leaves (>= 1) */
  int32_t reduce_op;      /* DG_OP_SUM or DG_OP_SUMSQ (fma: fused square-add) */
  int32_t split_layout;   /* DG_SPLIT_CONTIGUOUS: part s is the k range between
                             cuts s and s+1; DG_SPLIT_STRIDED: the K axis is
                             dealt in tiles of split_tile, tile u (k in
                             [u w, u w + w)) going to part u mod S, each part
                             walking its tiles in increasing k (Sec. 3.2.2, the
                             cut's layout).  A part may be empty (K < S w): its
                             value is +0.  Requires n_cuts = 0, tail =
                             DG_TAIL_LAST and split_tile a multiple of tile_k */
  int32_t split_tile;     /* w, the dealt tile (strided layout; else 0) */
  int32_t leaf_layout;    /* row reduction.  DG_LEAF_CONTIGUOUS: leaf j is the
                             elements [j leaf_w, (j+1) leaf_w).  DG_LEAF_STRIDED:
                             leaf_w leaves (lanes), leaf j folding elements j,
                             j + leaf_w, j + 2 leaf_w, ... in index order (Sec.
                             3.2.2 GEMV: lanes take every count-th element);
                             this build realises leaf_w a power of two <= 256 */
  int32_t lane_fold;      /* row reduction.  DG_FOLD_UP: the leaves meet in the
                             balanced tree in leaf order (a butterfly whose
                             offsets count up: the order Sec. 5.1 pins).
                             DG_FOLD_DOWN: the balanced tree over the leaf_w
                             lanes in bit-reversed order (a butterfly counting
                             its offsets down, the default of common kernels,
                             Sec. 3.2.2 GEMV); strided layout only.  An empty
                             lane (leaf_w > cols) joins no addition */
  int32_t norm_round;     /* dg_rmsnorm.  DG_NORM_FINAL: the normalised value
                             meets the weight at binary32; DG_NORM_PRE_WEIGHT:
                             it is rounded to bf16 first (an unfused "normalise
                             in fp32, cast to bf16, scale by the bf16 weight"
                             pair) */
  int32_t in_dtype;       /* GEMM operands A and B.  DG_IN_BF16 (default) or
                             DG_IN_F16: IEEE binary16, folded by the fp16
                             instruction of the same shape, whose chunks follow
                             the same rules with binary16 exponents (a product
                             of two binary16 values is exact in binary32, so the
                             scalar path is unchanged).  DG_IN_BF16_E4M3: A
                             bf16, B one byte per element in the OCP 8-bit
                             e4m3 format (bias 7, no infinities, S.1111.111
                             NaN), each value widened exactly to bf16 (every
                             e4m3 value is one) and folded by the bf16
                             instruction: the order and bits of a bf16 GEMM on
                             the widened B (the fp8 instructions fold
                             differently).  An e4m3 B is taken by the bf16 MFMA
                             descriptors only (not DG_MMA_SCALAR_FMA).
                             DG_IN_E4M3: A and B both one OCP e4m3 byte per
                             element, folded by the fp8 instruction the
                             descriptor names (it must name one of the
                             DG_MMA_*_FP8 / _F8F6F4 shapes, and they take no
                             other operands: DG_ERR_INVALID otherwise).  The
                             bias stays bf16. */
} dg_desc_params;

typedef struct dg_desc dg_desc; /* opaque, immutable */

/* Validate `p` and build an immutable descriptor.  *out receives a handle
 * owned by the caller (free with dg_desc_destroy).  Errors: DG_ERR_INVALID
 * (NULL arguments, struct_size too small, a field out of range),
 * DG_ERR_UNSUPPORTED (merge at bf16 over fp32 partials, pre-activation
 * rounding without an activation). */
dg_status dg_desc_create(const dg_desc_params* p, dg_desc** out);

/* Free a descriptor (NULL is ignored).  Calls already enqueued with it are
 * unaffected: launches copy what they need. */
void dg_desc_destroy(dg_desc* d);

/* Canonical text of the order a descriptor fixes (Sec. 4: the reconstructed
 * order is kept as a frozen record of every factor), NUL-terminated into buf
 * (capacity n).  Every field that can change a bit is written in full,
 * explicit cuts included, so descriptors with equal signatures give equal
 * bits; fields that cannot change bits (the instruction shape when fma = 1)
 * are normalised away.  The text is at most DG_SIGNATURE_MAX bytes with its
 * terminating NUL.  DG_ERR_INVALID if d or buf is NULL or buf is too small
 * (nothing is written then). */
dg_status dg_desc_signature(const dg_desc* d, char* buf, size_t n);

/* C = epilogue(A . B) in the descriptor's order: per output, the K axis cut
 * into parts, each part into tiles and instruction groups, the groups folded
 * into an accumulator (Sec. 3.2.1), the tiles and parts combined as the
 * descriptor says, the parts merged at merge_dtype (Sec. 3.2.2), then the
 * epilogue at its fixed rounding points (Sec. 1).
 *   A: device, M x K row-major;  B: device, K x N row-major; both bf16, or
 *   binary16 when in_dtype = DG_IN_F16;
 *   bias: device, N bf16, required iff the epilogue uses it (else ignored);
 *   C: device, M x N of out_dtype, row-major (written, never read).
 * M = 0 or N = 0 is a no-op returning DG_OK.  K = 0 is allowed when
 * split_k = 1 (every sum is +0).  DG_ERR_SHAPE if the plan for K leaves a
 * part empty or an explicit cut lies outside (0, K); DG_ERR_ALIGN if A, B,
 * bias or C is not aligned to its element size.  Split-K (S > 1) writes fp32
 * or bf16 partials to a library-owned workspace cached per (device, stream)
 * and merges them in a second kernel on the same stream (no atomics);
 * DG_ERR_NOMEM if that workspace cannot grow. */
dg_status dg_gemm(const dg_desc* d, const void* A, const void* B, const void* bias,
                  void* C, int64_t M, int64_t N, int64_t K, void* stream);

/* dg_gemm for callers that cannot allocate device memory (code under HIP
 * graph capture, tight serving loops, harnesses that forbid allocation):
 * the same kernels and the same bits as dg_gemm, but split-K partials
 * (S > 1) go to a fixed array of DG_NOALLOC_SCRATCH_BYTES (16 MiB) that the
 * library holds on each device it runs on until the process ends, instead of
 * the workspace dg_gemm grows.  The call allocates and frees nothing (no
 * hipMalloc, no hipFree, no allocating library routine); the caller passes
 * inputs and outputs as for dg_gemm.  DG_ERR_SCRATCH, before any launch, if
 * S * M * N * 4 bytes exceed the array (S = 1 uses no scratch).  Every call on
 * a device shares that device's one array, which keeps the last call's
 * partials: calls that overlap in time on one device (other streams, other
 * host threads) race and give undefined results; calls ordered on one stream
 * are safe.  Every partial a call reads was written by the same call, so
 * nothing needs clearing.  Errors otherwise as dg_gemm. */
dg_status dg_gemm_noalloc(const dg_desc* d, const void* A, const void* B, const void* bias,
                          void* C, int64_t M, int64_t N, int64_t K, void* stream);

/* Packed B for few-row GEMMs (a layout for the memory system; the order,
 * and so every bit, is the descriptor's, as Sec. 5.2 has it for layouts
 * under a pinned order).  Every 32 x 16 block of B (32 consecutive k of 16
 * consecutive columns) is one contiguous 1 KB run holding, for l = 0 .. 63
 * in turn, the 8 values B[k0 + 8 (l / 16) + e][n0 + l % 16], e = 0 .. 7 --
 * the B operand layout of the 16x16x32 MFMA -- and the runs are ordered by
 * column panel (n0 / 16), then by k block (k0 / 32).  Columns past N and k
 * past K are zeros.  The element type is not read (bf16 or binary16 alike).
 * dg_packed_b_bytes gives the size: ceil(N / 16) * ceil(K / 32) * 1024
 * bytes (0 for K = 0 or N = 0; SIZE_MAX for a negative size). */
size_t dg_packed_b_bytes(int64_t K, int64_t N);

/* The packed form of an e4m3 B (DG_IN_BF16_E4M3), one byte per element:
 * every 64 x 16 block (two 32-k blocks) is one 1 KB run, for l = 0 .. 63 in
 * turn the 8 bytes B[k0 + 8 (l / 16) + e][n0 + l % 16] of the first block
 * and then the 8 of the second (k0 + 32), so one 16-byte load per lane
 * brings a lane its operands of both blocks; runs by column panel, then by
 * k0 / 64; zeros past N and K.  dg_packed_b8_bytes: ceil(N / 16) *
 * ceil(K / 64) * 1024 (SIZE_MAX as dg_packed_b_bytes); dg_pack_b8 writes it
 * from a row-major K x N byte matrix, with the errors of dg_pack_b (B needs
 * no alignment). */
size_t dg_packed_b8_bytes(int64_t K, int64_t N);
dg_status dg_pack_b8(const void* B, void* Bp, int64_t K, int64_t N, void* stream);

/* Write the packed form of B (device, K x N row-major 16-bit elements) into
 * Bp (device, dg_packed_b_bytes(K, N) bytes, 16-byte aligned), on stream.
 * DG_ERR_SHAPE for a negative size; DG_ERR_ALIGN if B is not 2-byte or Bp
 * not 16-byte aligned; DG_ERR_INVALID for a NULL pointer with a non-empty
 * size.  One launch, no workspace. */
dg_status dg_pack_b(const void* B, void* Bp, int64_t K, int64_t N, void* stream);

/* dg_gemm with B in the packed form (Bp from dg_pack_b for the same K, N, or
 * dg_pack_b8 for a DG_IN_BF16_E4M3 descriptor):
 * the same order and the same bits as dg_gemm on the row-major B, on a
 * kernel that streams each 1 KB run with one coalesced load (one wave per
 * 16 columns, split-K part and up to 64 rows of A).  For few-row products:
 * M <= 64.  Descriptors: carried accumulator (tile_combine CARRY), fma 1,
 * no leading short tile; contiguous parts whose interior cut points are
 * multiples of 32 (64 for an e4m3 B), or strided parts dealing tiles of
 * 32 * 2^j k (64 * 2^j for an e4m3 B).
 * DG_ERR_UNSUPPORTED for anything else (M > 64 included), DG_ERR_ALIGN if Bp
 * is not 16-byte aligned; errors otherwise as dg_gemm.  Split-K uses the
 * same workspace, or none where two to eight contiguous parts meet in the
 * kernel (one launch). */
dg_status dg_gemm_packed(const dg_desc* d, const void* A, const void* Bp, const void* bias,
                         void* C, int64_t M, int64_t N, int64_t K, void* stream);

/* dg_gemm followed by the column sums of its output, an epilogue reduction
 * (the paper times a GEMM whose epilogue emits a column sum, Sec. 7):
 * colsum[j] = the balanced tree over the rows of column j in order (count
 * up; equal to the perfect tree over the rows padded to a power of two, the
 * padding taking no part), each output taken as stored (a bf16 output
 * widened exactly).  C is written exactly as dg_gemm writes it.
 *   colsum: device, N fp32 (written).  M = 0 gives +0 sums; N = 0 is a
 *   no-op.  Aligned runs of 256 rows are folded in parallel and their roots
 *   combined, through a library-owned workspace of ceil(M / 256) x N fp32
 *   values per (device, stream) when M > 256.  Errors as dg_gemm, plus
 *   DG_ERR_INVALID for a NULL colsum, DG_ERR_ALIGN for a misaligned one,
 *   DG_ERR_SHAPE for M > 65535 * 256. */
dg_status dg_gemm_colsum(const dg_desc* d, const void* A, const void* B, const void* bias,
                         void* C, float* colsum, int64_t M, int64_t N, int64_t K, void* stream);

/* Sizes and alignment (dg_gemm): bf16 and binary16 operands run on the tiled
 * kernels at any N, K >= 8, any part start and any element-aligned pointers
 * (small products off the 8-element grid whose parts are one slab, on the
 * generic kernel); strided splits, scalar descriptors and a short leading tile
 * off the chunk grid keep the kernels named below. */

/* Speed knobs for dg_gemm_knobs.  Any value gives the same bits as
 * dg_gemm; they exist so that this can be checked.  0 = the library's
 * choice. */
typedef struct {
  int32_t kernel;  /* 0 auto, 1 generic chunk-ordered kernel, 2 tiled MFMA kernel,
                      3 tiled MFMA kernel with transposing LDS reads and a
                      two-slab prefetch, 4 few-row kernel (tile_m <= 64,
                      tile_n 16/32/64) with a deep load ring, 5 eight-wave
                      ping-pong kernel (tile_m, tile_n each 128 or 256): two
                      groups of four waves one phase apart, 6 the kernel-5
                      256 x 256 blocks on the first split_n columns and
                      256 x 192 blocks on the rest, in one launch, 7 as 6 (or
                      256 x 256 blocks alone when split_n is 0 and no split
                      helps) with direct-to-LDS loads, 8 the few-row kernel with
                      a ring of depth (0 = 8) LDS slots filled by direct-to-LDS
                      loads (tile_m 0 = 16, tile_n 0 = 16, slab_k 0 = 256),
                      9 the scalar-FMA kernel, the only one for DG_MMA_SCALAR_FMA
                      descriptors (no other knob), 10 four waves with 128-row
                      sub-tiles and direct-to-LDS loads into a four-slot ring,
                      256 x 256 blocks on the first split_n columns and
                      256 x 192 blocks on the rest, 11 the packed-B kernel
                      (dg_gemm_packed only, which runs nothing else; tile_m
                      0, 16, 32 or 64 rows per wave, depth its ring of k
                      blocks), 12 the tile-combine kernel: tile_combine
                      DG_SEQ or DG_TREE, or fma = 0, on 128 x 64 blocks of
                      four waves (no other knob; K and N multiples of 8, the
                      operands 16-byte aligned, every part's tile boundaries
                      on 32-k steps from its start, fma = 0 only with the
                      16x16x32 instruction, a tree part at most 128 tiles,
                      otherwise DG_ERR_UNSUPPORTED; the library's choice
                      there for fma = 0, and for fma = 1 where a tree of nine
                      to sixteen tiles takes fewer rounds of the chip on it;
                      else kernel 0 runs smaller blocks that have no knob, on
                      any size of at least 8 and any alignment and up to 256
                      tiles).  Binary16 operands
                      (in_dtype = DG_IN_F16) run on kernels 0, 1, 3, 4, 5, 6,
                      9 and 12; kernels 2, 7, 8 and 10 return DG_ERR_UNSUPPORTED.
                      An e4m3 B (DG_IN_BF16_E4M3) runs on kernel 1 (row-major)
                      and kernel 11 (packed).  13 the fp8 kernel, the only one
                      besides kernel 1 for e4m3 x e4m3 (DG_IN_E4M3) and for
                      nothing else: four waves on the block-scaled fp8
                      instructions, blocks tile_m x tile_n of 128 x 128,
                      256 x 256 or 256 x 128 (0: 256 x 128 from 129 rows
                      on, else 128 x 128; no other knob); taken
                      when tile_combine is DG_CARRY,
                      fma = 1, the split contiguous, K and N multiples of
                      16, every part start and leading short tile on a
                      multiple of 16, A, B, C and bias 16-byte aligned;
                      otherwise DG_ERR_UNSUPPORTED, and kernel 0 runs the
                      generic kernel 1 (where it is taken, kernel 0 also has
                      smaller blocks without a knob).  e4m3 x e4m3 is not taken by
                      dg_gemm_packed.  14 bf16 operands on kernel 13's
                      pipeline (256 x 128 blocks, two per CU, 32x32x16
                      instructions; the tiled layout's conditions; no
                      other knob) */
  int32_t tile_m;  /* tiled kernels' rows per workgroup: 0, 16, 32, 64, 128, 256
                      (kernel 3: no 256 x 256 block) */
  int32_t tile_n;  /* tiled kernels' columns per workgroup: 0, 64, 128, 256 */
  int32_t order;   /* kernels 3, 5, 6, 7, 10: block order: 0 library's choice, 1 row-major
                      (consecutive workgroups share an A panel), 2 groups of
                      eight block rows walked column by column, 3 as 2 with
                      each of the eight XCDs given a contiguous range */
  int32_t occupancy; /* kernel 3: 0 library's choice, 1 or 2 workgroups per CU */
  int32_t depth;   /* kernel 4: slabs of loads kept in flight (0 = 4; 2, 4 or 8);
                      kernel 8: LDS ring slots; kernel 11: k blocks in flight
                      (16-row waves 8, 16, 24, 32; 32-row 8, 12, 16; 64-row
                      6, 10; with A rows not 16-byte aligned 4, 2, 1) */
  int32_t slab_k;  /* kernel 4: k per slab (0 = 64; 64, 128 or 256).  Kernel 4
                      builds a fixed list of (tile_m, tile_n, depth, slab_k);
                      others return DG_ERR_UNSUPPORTED */
  int32_t split_n; /* kernels 6, 7, 10: columns computed in 256-wide blocks, a multiple
                      of 256 in [0, N] (0 = library's choice, which may be 0:
                      all blocks 192 wide); tile_m, tile_n must be 0 */
} dg_knobs;

/* dg_gemm with explicit speed knobs (NULL = dg_gemm).  A knob combination
 * the build lacks returns DG_ERR_UNSUPPORTED before any launch. */
dg_status dg_gemm_knobs(const dg_desc* d, const void* A, const void* B, const void* bias,
                        void* C, int64_t M, int64_t N, int64_t K,
                        const dg_knobs* knobs, void* stream);

/* dg_gemm_packed with explicit speed knobs (kernel 0 or 11, tile_m, depth;
 * every other knob 0). */
dg_status dg_gemm_packed_knobs(const dg_desc* d, const void* A, const void* Bp, const void* bias,
                               void* C, int64_t M, int64_t N, int64_t K,
                               const dg_knobs* knobs, void* stream);

/* out[r] = balanced-tree reduction of row r of X (Sec. 3.1, Sec. 5.1):
 * leaves of leaf_w consecutive elements folded in index order (SUM: s = x0,
 * s (+)= xi; SUMSQ: s = RN32(x0^2), then fma(xi, xi, s) if fma = 1 else
 * s (+) RN32(xi^2)), then the leaves combined by the balanced tree (pairs of
 * neighbours level by level, an odd last leaf carried up).
 *   X: device, rows x cols fp32 row-major;  out: device, rows fp32.
 * rows = 0 is a no-op; cols = 0 writes +0 to every out[r].  DG_ERR_ALIGN if
 * X or out is not 4-byte aligned. */
dg_status dg_rowsum(const dg_desc* d, const float* X, float* out, int64_t rows,
                    int64_t cols, void* stream);

/* Root-mean-square normalisation of each row, on the row's sum of squares
 * in the descriptor's order (exactly the value dg_rowsum returns for the
 * descriptor with reduce_op DG_OP_SUMSQ: leaf_w, leaf_layout, lane_fold and
 * fma apply; the descriptor's reduce_op must be DG_OP_SUMSQ).  Then, each
 * step one IEEE binary32 operation (sqrt and division correctly rounded):
 *   ms = s / n (n = cols as binary32),  v = ms + eps,  q = sqrt(v),
 *   rinv = 1 / q,  y_j = x_j * rinv,
 *   y'_j = y_j (DG_NORM_FINAL) or RN_bf16(y_j) (DG_NORM_PRE_WEIGHT),
 *   out_j = RN_out(y'_j * w_j), or RN_out(y'_j) when w is NULL.
 * These are the steps around the pinned reduction that normalisation kernels
 * run (the paper's evaluation, Sec. 7: rmsnorm).
 *   X: device, rows x cols fp32 row-major;  w: device, cols bf16 or NULL;
 *   Y: device, rows x cols of out_dtype (written, never read; may not
 *   overlap X).  rows = 0 or cols = 0 is a no-op.  One launch (always under
 *   capture where one can serve the order), or two on `stream` through a library-owned workspace of rows fp32 values per
 *   (device, stream) (DG_ERR_NOMEM if it cannot grow).  Errors as dg_rowsum, plus
 *   DG_ERR_INVALID for a descriptor whose reduce_op is not DG_OP_SUMSQ. */
dg_status dg_rmsnorm(const dg_desc* d, const float* X, const void* w, float eps, void* Y,
                     int64_t rows, int64_t cols, void* stream);

/* Layer normalisation of each row in the centred form, both row sums in the
 * descriptor's leaf order (leaf_w, leaf_layout, lane_fold; the squares by
 * its fma rule; reduce_op is not used):
 *   s1 = the sum of x_j,  mean = s1 / n (n = cols as binary32),
 *   d_j = x_j - mean,  s2 = the sum of squares of the d_j,
 *   v = s2 / n + eps,  rinv = 1 / sqrt(v),  y_j = d_j * rinv,
 *   y'_j = y_j (DG_NORM_FINAL) or RN_bf16(y_j) (DG_NORM_PRE_WEIGHT),
 *   out_j = RN_out((y'_j * w_j) + b_j),
 * each step one IEEE binary32 operation; w and b (device, cols bf16 each)
 * are optional (NULL leaves the step out).  The paper evaluates layernorm
 * kernels (Sec. 7); the two sums are the order-sensitive steps.
 *   X: device, rows x cols fp32;  Y: device, rows x cols of out_dtype (may
 *   not overlap X).  rows = 0 or cols = 0 is a no-op.  One launch for
 *   contiguous leaves of 64 and strided lanes (64, 128 or 256) with fma = 1
 *   where that is the faster way, under capture, or where the other way would
 *   hold over 256 MB, up to 8388608 columns; otherwise four launches through a library-owned workspace of rows x (cols + 2) fp32
 *   values per (device, stream).  Errors as dg_rowsum. */
dg_status dg_layernorm(const dg_desc* d, const float* X, const void* w, const void* b, float eps,
                       void* Y, int64_t rows, int64_t cols, void* stream);

/* Softmax of each row, the row sum in the descriptor's order (exactly the
 * value dg_rowsum returns for the descriptor with reduce_op DG_OP_SUM:
 * leaf_w, leaf_layout and lane_fold apply; reduce_op must be DG_OP_SUM):
 *   m = max_j x_j (a NaN anywhere gives NaN; a maximum has no rounding, so
 *   its order is free),  e_j = exp(x_j - m) by the library's own binary32
 *   exp (the one of the SiLU epilogue: Cody-Waite reduction, degree-7
 *   Taylor polynomial, exact power-of-two scaling),  s = the sum of the e_j,
 *   rinv = 1 / s,  out_j = RN_out(e_j * rinv)  (each step one binary32
 *   operation).  The paper evaluates softmax kernels (Sec. 7); the sum is
 *   the only order-sensitive step.
 *   X: device, rows x cols fp32 row-major;  Y: device, rows x cols of
 *   out_dtype (written, never read; may not overlap X).  rows = 0 or
 *   cols = 0 is a no-op.  One launch when the descriptor has contiguous
 *   leaves of 64 or strided lanes (64, 128 or 256) where that is the faster
 *   way, under capture, or where the other way would hold over 256 MB, up to
 *   8388608 columns; fewer than 256 rows of 65537 to 262144 columns
 *   over contiguous leaves take three launches and a small workspace, anything
 *   else three launches through a library-owned workspace of rows x (cols + 1)
 *   fp32 values per (device, stream) (DG_ERR_NOMEM if it cannot grow).  Errors as dg_rowsum, plus DG_ERR_INVALID for a
 *   descriptor whose reduce_op is not DG_OP_SUM. */
dg_status dg_softmax(const dg_desc* d, const float* X, void* Y, int64_t rows, int64_t cols,
                     void* stream);

/* ------------------------------------------------------------- attention
 *
 * The reduction order of one attention head (App. F).  Per query row the
 * keys are walked in blocks; the row carries a running maximum m, a
 * denominator l and an output row O in binary32, starting from m = -inf,
 * l = +0, O = +0.  At a block of keys kb .. ke-1:
 *   s_t   = RN32(score_t * qk_scale), score_t = q . k_t over the head
 *           dimension in groups of 32 (the 16x16x32 instruction, chunks of 8
 *           in increasing order) from +0; under a causal mask a key above the
 *           diagonal in the masked stage gets s_t (+) -1e6 (its probability
 *           underflows to zero);
 *   mn    = max(m, max_t s_t);  alpha = exp2(m - mn);  p_t = exp2(s_t - mn),
 *           exp2 the library's own binary32 base-two exponential (Cody-Waite
 *           style split x = n + f, degree-7 polynomial for 2^f, exact scaling);
 *           the caller folds log2 e into qk_scale;
 *   rs    = the block's p_t summed in the order block_sum names: DG_SEQ, a
 *           chain in key order, or DG_TREE, the balanced tree over the
 *           block's positions in key order;
 *   l     = RN32(alpha l) (+) rs, or fma(alpha, l, rs) when l_fma;
 *   O_c   = P~ . V over the block's keys in groups of 32 from the block start,
 *           P~ = p narrowed to p_dtype before it meets V, with RN32(alpha O_c)
 *           as the accumulator (pv_fma) or from +0 and then added to it;
 *   m     = mn.
 * The answer is O_c / l per element, or O_c * RN32(1 / l) (final), rounded
 * to out_dtype.  The blocks: unmasked, width key_block from key 0 (the last
 * one shorter); causal (key t visible to query i iff t <= i, Lq = Lk), with
 * q0 = (i / q_block) q_block and q1 = min(q0 + q_block, Lk): [0, q0) cut into
 * blocks of key_block from key 0, the last ending at q0, then [q0, q1) cut
 * into blocks of key_block from q0, the last ending at q1, in which the keys
 * above the diagonal are masked.  So q_block (BLOCK_M) takes part in a
 * causal answer whenever it is not a multiple of key_block. */
enum { DG_ATTN_DIV = 0, DG_ATTN_RECIP = 1 };

typedef struct {
  uint32_t struct_size;   /* sizeof(dg_attn_params) */
  int32_t key_block;      /* w, keys per block (BLOCK_N), >= 1 */
  int32_t causal;         /* 0: no mask; 1: causal (Lq = Lk) */
  int32_t q_block;        /* BLOCK_M, >= 1: where the masked stage starts (causal) */
  int32_t block_sum;      /* DG_SEQ or DG_TREE: the row sum of a block's probabilities */
  int32_t p_dtype;        /* DG_BF16: the type the probabilities are narrowed to */
  int32_t pv_fma;         /* 1: the rescaled output row is the P.V accumulator */
  int32_t l_fma;          /* 1: the denominator update is one fused multiply-add */
  int32_t final_div;      /* DG_ATTN_DIV: O / l;  DG_ATTN_RECIP: O * (1 / l) */
  int32_t out_dtype;      /* DG_F32 or DG_BF16 */
} dg_attn_params;

typedef struct dg_attn_desc dg_attn_desc; /* opaque, immutable */

/* Validate p and build an attention descriptor (free with
 * dg_attn_desc_destroy).  DG_ERR_INVALID for NULL arguments, a small
 * struct_size or a field out of range; DG_ERR_UNSUPPORTED for an order this
 * build cannot run: key_block other than 32, 64 or 128, p_dtype other than
 * bf16, or a causal q_block that is not a multiple of 16. */
dg_status dg_attn_desc_create(const dg_attn_params* p, dg_attn_desc** out);
void dg_attn_desc_destroy(dg_attn_desc* d);

/* O = attention(Q, K, V) in the descriptor's order, for H independent heads.
 *   Q: device, H x Lq x d bf16;  K, V: device, H x Lk x d bf16;  O: device,
 *   H x Lq x d of out_dtype (written, never read); all row-major and 16-byte
 *   aligned.  d is 64 or 128.  qk_scale multiplies each score (fold log2 e
 *   and 1 / sqrt(d) into it).
 * H = 0 or Lq = 0 is a no-op.  DG_ERR_SHAPE for Lk < 1, H > 65535,
 * Lq > 16 * 65535, or a causal descriptor with Lq != Lk; DG_ERR_UNSUPPORTED for another d;
 * DG_ERR_ALIGN for a pointer not 16-byte aligned.  One launch on stream; for
 * few query rows over many keys three launches through a library-owned
 * workspace of the (device, stream), attention's own (at most 320 MB; never
 * while the stream is captured, and one launch again if it cannot grow). */
dg_status dg_attention(const dg_attn_desc* d, const void* Q, const void* K, const void* V, void* O,
                       int64_t H, int64_t Lq, int64_t Lk, int64_t dim, float qk_scale, void* stream);

/* Static text for a status code (never NULL; unknown codes give
 * "unknown status"). */
const char* dg_strerror(dg_status s);

/* Library version (major * 10000 + minor * 100 + patch).  0.2.0 (200) added
 * dg_desc_params.leaf_layout / lane_fold and dg_knobs.split_n: a caller
 * built against an earlier header must not pass its dg_knobs to this one.
 * 0.3.0 (300) added dg_desc_params.in_dtype (a smaller struct_size is
 * rejected) and knob kernel 10.  0.4.0 (400) added dg_gemm_noalloc and
 * DG_ERR_SCRATCH, and the attention descriptor and dg_attention.  0.5.0
 * (500) added the packed B form (dg_packed_b_bytes, dg_pack_b,
 * dg_gemm_packed, dg_gemm_packed_knobs), knob kernel 11, and e4m3 weights
 * (DG_IN_BF16_E4M3, dg_packed_b8_bytes, dg_pack_b8).  0.5.1 (501) added knob
 * kernel 12 (tile chain and tree, fma = 0, on a tiled kernel).  0.6.0 (600)
 * added e4m3 x e4m3 (DG_IN_E4M3, the DG_MMA_*_FP8 and _F8F6F4
 * instructions) and knob kernel 13. */
int32_t dg_version(void);

#ifdef __cplusplus
}
#endif
#endif /* DG_H */
