// Plain-data kernel argument records and the kernel list, shared by the host-side
// planner (which fills them at DAG build time) and the HIP translation unit (which
// launches them).  No HIP types here: the planner builds without a GPU toolchain.
#pragma once
#include <stdint.h>

namespace opara {

// Implicit-GEMM convolution / GEMM / strided batched GEMM.
//   D[n][m] = alpha * sum_k Wt[n][k] * Xg[m][k]   (n: output channel/column, m: pixel/row)
// Xg is either a plain matrix (gather == 0, row stride lda) or an on-the-fly patch
// gather from an [H][W][Cin] image with k = (i*kw + j)*Cin + ci (gather == 1).
struct IgemmArgs {
  const void *x, *w;
  const float *bias;
  void *y;
  const void *extra[3];
  int32_t n_extra;
  int32_t M, N, K;
  int32_t gather;
  int32_t H, W, Cin, Wo, kh, kw, sh, sw, ph, pw;
  int32_t HoWo;                 // output pixels per image; row m belongs to image m / HoWo
  int64_t img_stride;           // elements between consecutive input images (H*W*Cin)
  int64_t lda, ldb, ldy;        // row strides in elements
  int64_t a_bs, b_bs, y_bs;     // batch strides in elements (blockIdx.z)
  int32_t b_kmajor;             // second operand stored [K][N]
  int32_t relu;
  float alpha;
  uint32_t div_HoWo, div_Wo, div_Cin, div_kw;   // min(2^32 / d, 2^32 - 1): see fast_div
  uint32_t x_bytes, w_bytes;    // what the operands span (one batch element), 0 if one of them kOperandMaxBytes or more
  uint32_t div_gx;              // reciprocal of the grid's width
};

struct PoolArgs {
  const void *x;
  void *y;
  int32_t H, W, C, Ho, Wo, kh, kw, sh, sw, ph, pw;
  int32_t is_avg;
  int32_t B;                    // images
  uint32_t items;               // output pixels x channel chunks; 0: more than 32-bit byte offsets reach
  uint32_t div_cch, div_Wo, div_HoWo;   // reciprocals for fast_div
};

struct GapArgs {
  const void *x;
  void *y;
  int32_t HW, C;              // per image; blockIdx.y is the image
  int32_t vec;                // 16-byte chunks, two threads per pixel (1 << kGapShare)
};

struct RowArgs {               // LayerNorm / softmax over rows of the summed inputs
  const void *in[8];
  void *y;
  int32_t n_in, rows, cols;
  float eps;
};

struct EltArgs {               // f(sum of inputs), f in {identity, relu, gelu}
  const void *in[8];
  void *y;
  int32_t n_in, op;            // op: 0 add, 1 relu, 2 gelu
  int64_t n;
  // The result once more, as also_cols columns of rows also_pitch apart: the place of this
  // operator's result in a concatenation (fused executor, vector form); null: nowhere.
  void *also;
  int32_t also_cols, also_pitch;
  uint32_t div_also;           // reciprocal of the chunks per row
};

struct ConcatArgs {
  const void *in[8];
  void *y;
  int32_t cols[8], col_off[8];
  uint32_t div_cols[8];         // reciprocals of the chunks per row
  int32_t n_in, rows, out_cols;
};

// Scores, softmax and context of one attention in one launch (fused executor); z: head.
//   s[z] = alpha_s * q[z] . k[z]^T,  p[z] = softmax(s[z]),  y[z] = alpha_c * p[z] . v[z]
struct AttnArgs {
  const void *q, *k, *v;
  void *s, *p, *y;              // s, p: [heads][M][N] without gaps
  int64_t q_bs, k_bs, v_bs, y_bs, ldy;
  int32_t ldq, ldk, ldv;
  int32_t M, N, D, D2;          // query rows, key rows, width of a row of q and k, of v
  uint32_t q_bytes, k_bytes, v_bytes;   // one head
  float alpha_s, alpha_c;
  uint32_t div_gx;              // reciprocal of the grid's width
};

// X(name, ArgsType).  Order defines kernel ids.
#define OPARA_KERNEL_LIST(X)            \
  X(igemm_f16_t128x64, IgemmArgs)       \
  X(igemm_f16_tile64x64, IgemmArgs)     \
  X(igemm_f16_tile128x128, IgemmArgs)   \
  X(igemm_f16_t64x64, IgemmArgs)        \
  X(igemm_f16_direct4, IgemmArgs)       \
  X(igemm_f16_quad4, IgemmArgs)         \
  X(igemm_f16_quad64x4, IgemmArgs)      \
  X(igemm_f16_quad64x64, IgemmArgs)     \
  X(igemm_f16_t64x64_scalar, IgemmArgs) \
  X(igemm_f32_t128x64, IgemmArgs)       \
  X(igemm_f32_tile64x64, IgemmArgs)     \
  X(igemm_f32_tile128x128, IgemmArgs)   \
  X(igemm_f32_t64x64, IgemmArgs)        \
  X(igemm_f32_direct4, IgemmArgs)       \
  X(igemm_f32_quad4, IgemmArgs)         \
  X(igemm_f32_quad64x4, IgemmArgs)      \
  X(igemm_f32_quad64x64, IgemmArgs)     \
  X(igemm_f32_t64x64_scalar, IgemmArgs) \
  X(gemv_f16, IgemmArgs)                \
  X(gemv_f32, IgemmArgs)                \
  X(pool_f16_vec, PoolArgs)             \
  X(pool_f16_scalar, PoolArgs)          \
  X(pool_f32_vec, PoolArgs)             \
  X(pool_f32_scalar, PoolArgs)          \
  X(gap_f16, GapArgs)                   \
  X(gap_f32, GapArgs)                   \
  X(layernorm_f16_wave, RowArgs)        \
  X(layernorm_f16_block, RowArgs)       \
  X(layernorm_f16_generic, RowArgs)     \
  X(layernorm_f32_wave, RowArgs)        \
  X(layernorm_f32_block, RowArgs)       \
  X(layernorm_f32_generic, RowArgs)     \
  X(softmax_f16_wave, RowArgs)          \
  X(softmax_f16_block, RowArgs)         \
  X(softmax_f16_generic, RowArgs)       \
  X(softmax_f32_wave, RowArgs)          \
  X(softmax_f32_block, RowArgs)         \
  X(softmax_f32_generic, RowArgs)       \
  X(elt_f16_vec, EltArgs)               \
  X(elt_f16_scalar, EltArgs)            \
  X(elt_f32_vec, EltArgs)               \
  X(elt_f32_scalar, EltArgs)            \
  X(concat_f16_vec, ConcatArgs)         \
  X(concat_f16_scalar, ConcatArgs)      \
  X(concat_f32_vec, ConcatArgs)         \
  X(concat_f32_scalar, ConcatArgs)      \
  X(igemm_f16_direct4s, IgemmArgs)      \
  X(igemm_f16_quad4s, IgemmArgs)        \
  X(igemm_f32_direct4s, IgemmArgs)      \
  X(igemm_f32_quad4s, IgemmArgs)        \
  X(igemm_f16_far128x128, IgemmArgs)    \
  X(igemm_f32_far128x128, IgemmArgs)    \
  X(attention_f16, AttnArgs)            \
  X(igemm_f16_quad4s_tail, IgemmArgs) \
  X(igemm_f16_quad4_tail, IgemmArgs) \
  X(igemm_f16_quad64x4_tail, IgemmArgs) \
  X(igemm_f16_quad64x64_tail, IgemmArgs) \
  X(igemm_f16_tile64x64_tail, IgemmArgs) \
  X(igemm_f16_t128x64_tail, IgemmArgs) \
  X(igemm_f16_tile128x128_tail, IgemmArgs) \
  X(igemm_f32_quad4s_tail, IgemmArgs) \
  X(igemm_f32_quad4_tail, IgemmArgs) \
  X(igemm_f32_quad64x4_tail, IgemmArgs) \
  X(igemm_f32_quad64x64_tail, IgemmArgs) \
  X(igemm_f32_tile64x64_tail, IgemmArgs) \
  X(igemm_f32_t128x64_tail, IgemmArgs) \
  X(igemm_f32_tile128x128_tail, IgemmArgs)

enum KernelId : int32_t {
#define X(name, T) K_##name,
  OPARA_KERNEL_LIST(X)
#undef X
  K_COUNT
};

union KernelArgs {
  IgemmArgs igemm;
  PoolArgs pool;
  GapArgs gap;
  RowArgs row;
  EltArgs elt;
  ConcatArgs concat;
  AttnArgs attn;
};

// An element-wise operator computed by the contraction that produces one of its inputs (fused
// executor): y = f(sum of n_in inputs), all without gaps and of the contraction's size.
struct TailArgs {
  const void *in[2];            // the inputs that are not the contraction's result, in order
  void *y;
  int32_t n_in, self, op;       // self: place of the contraction's result among the inputs; op as in EltArgs
  int32_t reserved;
};

// Second argument of every planned kernel: the operator id, the grid and the operator-timeline
// buffer (null: off).
struct LaunchArgs {
  int32_t tag, gx, gy, gz;
  unsigned long long *trace;
};

// One planned launch: which kernel, its grid and its arguments.
struct KernelPlan {
  int32_t kernel;
  uint32_t gx, gy, gz;
  uint32_t block;
  int32_t tag;                  // operator id: slot of the operator timeline
  KernelArgs args;
  TailArgs tail;                // contractions with a tail only
};

// A group node: up to kGroupMaxOps mutually independent operators launched as ONE kernel
// whose grid is the sum of their grids.  Workgroup w serves the operator i with
// block_end[i-1] <= w < block_end[i]; each operator's range is padded to a multiple of the
// XCD count (padding workgroups leave at once), so that tile t of an operator runs on XCD
// t % 8 as in a launch of its own.  The record travels by value as the kernel argument.
constexpr int kGroupMaxOps = 16;
constexpr int kGroupAlign = 8;
struct GroupMeta {                                 // one member: read with one 32-byte scalar load
  int32_t kernel;                                  // KernelId of the operator's body
  int32_t gx, gy;                                  // the operator's own grid (x, y; z follows)
  int32_t tiles;                                   // gx * gy * gz
  int32_t tag;                                     // operator id (slot of the operator timeline)
  int32_t block_begin;                             // first block of the member's range
  uint32_t div_gx;                                 // reciprocal of gx for fast_div
  int32_t gz;
};
struct GroupArgs {
  int32_t block_end[kGroupMaxOps];
  int32_t n;
  int32_t reserved;
  unsigned long long *trace;                       // operator-timeline buffer, null = off
  GroupMeta meta[kGroupMaxOps];
  KernelArgs args[kGroupMaxOps];
};
// Operands of the LDS-fed contractions are addressed through 32-bit buffer offsets; this
// offset is past the end of every operand they accept, and stays so with a row of K added.
// Larger operands take a body of their own, which counts from the first row, or image, of its tile
// of kFarTile x kFarTile (fp16, 394,000 x 4096 x 512: 1.8 ms; register-staged, with 64-bit
// addresses, 6.5 ms).  Every body doing so costs the small networks 1.3 %.
constexpr uint32_t kOperandMaxBytes = 0xc0000000u;
constexpr int kFarTile = 128;

// Tile geometry of the implicit-GEMM kernels (output columns x rows per workgroup).
struct IgemmTile { int bn, bm; };
constexpr IgemmTile kTile128x64{128, 64};
constexpr double kTiledMinFlopsPersistent = 2.0e9;   // persistent kernel: lighter contractions use 32 x 32 tiles
constexpr int kTiledMinTiles = 80;               // ... and so do contractions with fewer 128x64 tiles
constexpr IgemmTile kTile64{64, 64};
constexpr int64_t kQuadMinRowBytes = 512;    // shorter rows of K stay on the fragment-loading kernels
constexpr int64_t kDirectMaxTiles32 = 512;  // ... unless there are so many tiles that bytes count, not latency
                                             // (three 1 x 1 convolutions of 16 images of 192 x 35 x 35: 20.8 -> 15.4 us)
constexpr int kDirectTile = 32;       // output tile edge of the fragment-loading kernels
constexpr int kSmallTile = 16;        // ... of their small-tile form, for operators with few 32 x 32 tiles
constexpr int kSmallTileMaxTiles32 = 100;   // at most this many 32 x 32 tiles: take 16 x 16 ones (four times as many workgroups)

constexpr int kRowGroupWave = 64;     // threads cooperating on one row (wave variant)
constexpr int kRowGroupBlock = 256;   // block variant
constexpr int kRowCacheChunks = 4;    // 16-byte chunks a thread keeps in registers
constexpr int kAttnMaxCols = 512;     // attention kernel: one 16-byte chunk of scores per lane of a wavefront
constexpr int kAttnMaxWidth = 64;     // ... one 128-byte line per row of q, k and v
constexpr int kGemvMaxM = 4;
constexpr int kGapShare = 1;          // global average: log2 of the threads that share a pixel (vector form)
constexpr int kGapVecMinPixels = 128; // ... taken from this many pixels on

}  // namespace opara
