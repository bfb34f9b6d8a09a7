// Kernel table and per-operator launch planning (host only, no HIP calls).
// The demand record of an operator (paper Sec. 3.2: threads, shared memory and
// registers of one block; Sec. 2.3: number of blocks) follows from the plan made
// here plus the static resources of the chosen kernel.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <tuple>
#include <vector>
#include "opara_internal.h"

namespace opara {

// Generated at build time from the compiler's per-kernel resource report of
// kernels.hip; one row per entry of OPARA_KERNEL_LIST, same order.
const KernelResource kKernelResources[K_COUNT] = {
#include "kernel_resources.inc"
};

namespace {

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline uint32_t cdiv(int64_t a, int64_t b) { return (uint32_t)((a + b - 1) / b); }

// The contractions fed through workgroup memory, and what one workgroup of each costs, in
// microseconds: a 128-byte step of K when the workgroup has a compute unit to itself
// (`alone`) and when the launch keeps every CU busy (`busy`), and everything outside the K
// walk (`fixed`).  `together`: how much longer the work takes inside a group kernel;
// fitted, like the rest (three 512 x 768 x 768 products: 8.3 -> 7.5 us with the tiles this makes
// them take).  Fitted to isolated fp16 products, M x N x K = 49..346688 x 32..4096 x
// 320..4096, within 15 %.  In fp32 a step cannot take less than its multiply-adds at the
// matrix rate of a CU (0.6 TFLOP/s).
struct TileKernel { int ids[2]; int bn, bm; double alone, busy, fixed, together; };   // ids: f32, f16
const TileKernel kTileKernels[] = {
    {{K_igemm_f32_quad4s, K_igemm_f16_quad4s}, 16, 16, 0.060, 0.037, 0.25, 1},
    {{K_igemm_f32_quad4, K_igemm_f16_quad4}, 32, 32, 0.080, 0.075, 0.58, 1},
    {{K_igemm_f32_quad64x4, K_igemm_f16_quad64x4}, 64, 32, 0.122, 0.125, 0.50, 1.15},
    {{K_igemm_f32_quad64x64, K_igemm_f16_quad64x64}, 64, 64, 0.160, 0.165, 1.6, 1.2},
    {{K_igemm_f32_tile64x64, K_igemm_f16_tile64x64}, 64, 64, 0.28, 0.18, 0.8, 1},
    {{K_igemm_f32_t128x64, K_igemm_f16_t128x64}, 128, 64, 0.45, 0.33, 1.2, 1},
    {{K_igemm_f32_tile128x128, K_igemm_f16_tile128x128}, 128, 128, 0.56, 0.48, 1.7, 1},
};
constexpr int kTileKernelCount = sizeof kTileKernels / sizeof kTileKernels[0];
constexpr double kCus = 256.0;
bool tile_kernel_is_f16(int id) {
  return std::any_of(kTileKernels, kTileKernels + kTileKernelCount, [&](const TileKernel &t) { return t.ids[1] == id; });
}

int fail(const char *what, const opara_op_desc &op) {
  set_error("operator type %d: %s", op.op_type, what);
  return OPARA_EINVAL;
}

int plan_igemm(const opara_op_desc &op, const void *const *in, int kind, KernelPlan *out) {
  const bool persistent = kind == kPlanPersistent;
  const opara_op_params &p = op.params;
  const bool f16 = op.dtype == OPARA_F16;
  const int ve = f16 ? 8 : 4;
  IgemmArgs a;
  std::memset(&a, 0, sizeof a);
  a.x = in[0];
  a.bias = op.bias;
  a.y = op.out;
  a.alpha = 1.0f;
  a.HoWo = a.Wo = a.Cin = a.kw = 1;
  a.relu = (p.flags & OPARA_FLAG_RELU) ? 1 : 0;
  int64_t batch = 1;
  bool vec;
  if (op.op_type == OPARA_CONV2D) {
    if (op.n_inputs != 1 || !op.weight) return fail("convolution needs one input and a weight", op);
    if (p.h_in <= 0 || p.w_in <= 0 || p.c_in <= 0 || p.c_out <= 0 || p.kh <= 0 || p.kw <= 0 ||
        p.sh <= 0 || p.sw <= 0 || p.ph < 0 || p.pw < 0)
      return fail("bad convolution geometry", op);
    if (p.h_out != (p.h_in + 2 * p.ph - p.kh) / p.sh + 1 || p.w_out != (p.w_in + 2 * p.pw - p.kw) / p.sw + 1 ||
        p.h_out <= 0 || p.w_out <= 0)
      return fail("convolution output size does not match floor((in + 2*pad - k)/stride) + 1", op);
    if (p.batch < 0 || p.batch > 4096) return fail("bad image batch", op);
    const int images = p.batch > 0 ? p.batch : 1;
    a.w = op.weight;
    a.HoWo = p.h_out * p.w_out;
    a.img_stride = (int64_t)p.h_in * p.w_in * p.c_in;
    a.M = images * a.HoWo;
    a.N = p.c_out;
    a.K = p.kh * p.kw * p.c_in;
    a.gather = !(p.kh == 1 && p.kw == 1 && p.sh == 1 && p.sw == 1 && p.ph == 0 && p.pw == 0);
    a.H = p.h_in; a.W = p.w_in; a.Cin = p.c_in; a.Wo = p.w_out;
    a.kh = p.kh; a.kw = p.kw; a.sh = p.sh; a.sw = p.sw; a.ph = p.ph; a.pw = p.pw;
    if (p.c_row_stride != 0 && p.c_row_stride < p.c_out) return fail("output pixel stride below c_out", op);
    a.lda = p.c_in; a.ldb = a.K; a.ldy = p.c_row_stride ? p.c_row_stride : p.c_out;
    vec = (p.c_in % ve == 0);
  } else if (op.op_type == OPARA_GEMM) {
    if (!op.weight || op.n_inputs > 4) return fail("GEMM needs a weight and at most 3 extra inputs", op);
    if (p.m <= 0 || p.n <= 0 || p.k <= 0) return fail("bad GEMM shape", op);
    a.w = op.weight;
    a.M = p.m; a.N = p.n; a.K = p.k;
    if (p.c_row_stride != 0 && p.c_row_stride < p.n) return fail("output row stride below n", op);
    a.lda = p.k; a.ldb = p.k; a.ldy = p.c_row_stride ? p.c_row_stride : p.n;
    a.HoWo = p.m; a.Wo = 1;
    a.n_extra = op.n_inputs - 1;
    for (int i = 0; i < a.n_extra; ++i) a.extra[i] = in[i + 1];
    vec = (p.k % ve == 0);
  } else {  // BGEMM
    if (op.n_inputs != 2) return fail("batched GEMM needs two inputs", op);
    if (p.m <= 0 || p.n <= 0 || p.k <= 0 || p.batch <= 0 || p.batch > 65535) return fail("bad batched GEMM shape", op);
    if (p.a_row_stride < p.k || p.c_row_stride < p.n || p.a_batch_stride < 0 || p.b_batch_stride < 0 ||
        p.c_batch_stride < 0)
      return fail("bad batched GEMM strides", op);
    a.w = in[1];
    a.M = p.m; a.N = p.n; a.K = p.k;
    a.lda = p.a_row_stride; a.ldb = p.b_row_stride; a.ldy = p.c_row_stride;
    a.HoWo = p.m; a.Wo = 1;
    a.a_bs = p.a_batch_stride; a.b_bs = p.b_batch_stride; a.y_bs = p.c_batch_stride;
    a.b_kmajor = (p.flags & OPARA_FLAG_B_KMAJOR) ? 1 : 0;
    if (a.b_kmajor ? p.b_row_stride < p.n : p.b_row_stride < p.k) return fail("bad batched GEMM strides", op);
    a.alpha = p.alpha;
    batch = p.batch;
    vec = (p.k % ve == 0) && (a.lda % ve == 0) && (a.ldb % ve == 0) && (a.a_bs % ve == 0) && (a.b_bs % ve == 0) &&
          (!a.b_kmajor || p.n % ve == 0);
  }
  vec = vec && aligned16(a.x) && aligned16(a.w);
  a.div_HoWo = div_magic(a.HoWo); a.div_Wo = div_magic(a.Wo);
  a.div_Cin = div_magic(a.Cin); a.div_kw = div_magic(a.kw);
  auto set = [&](int kernel, int bn, int bm) {
    out->kernel = kernel;
    out->gx = cdiv(a.M, bm);
    out->gy = cdiv(a.N, bn);
    out->gz = (uint32_t)batch;
    out->block = 256;
    a.div_gx = div_magic((int64_t)out->gx);
    out->args.igemm = a;
    return OPARA_OK;
  };
  if (vec && op.op_type == OPARA_GEMM && a.M <= kGemvMaxM) {
    set(f16 ? K_gemv_f16 : K_gemv_f32, 1, 1);
    out->gx = cdiv(a.N, 4);            // one wave per output column, four waves per workgroup
    out->gy = 1;
    return OPARA_OK;
  }
  if (!vec) return set(f16 ? K_igemm_f16_t64x64_scalar : K_igemm_f32_t64x64_scalar, kTile64.bn, kTile64.bm);
  const int64_t es = f16 ? 2 : 4;
  const int64_t x_bytes = es * (a.gather ? (int64_t)(a.M / a.HoWo) * a.img_stride : (int64_t)(a.M - 1) * a.lda + a.K);
  const int64_t w_bytes = es * ((int64_t)(a.N - 1) * a.ldb + a.K);
  const int64_t reach = kOperandMaxBytes;
  const bool fits = x_bytes < reach && w_bytes < reach;
  a.x_bytes = fits ? (uint32_t)x_bytes : 0;
  a.w_bytes = fits ? (uint32_t)w_bytes : 0;
  // What 32-bit offsets have to span inside one tile of larger operands.
  const int64_t tile_x = es * (a.gather ? (int64_t)(kFarTile / a.HoWo + 2) * a.img_stride : (int64_t)kFarTile * a.lda + a.K);
  const int64_t tile_w = es * ((int64_t)kFarTile * a.ldb + a.K);
  const bool far = !fits && tile_x < reach && tile_w < reach && !persistent;   // the persistent kernel does not hold that body
  const bool steps = a.K * es < (int64_t)1 << 29 && (!a.gather || ((int64_t)a.kh * a.W + a.kw < 1 << 24 && a.Cin < 1 << 24));
  // [K][N] operand, or out of the reach of 32-bit offsets: staged through registers.
  if (a.b_kmajor || !steps || !(fits || far))
    return set(f16 ? K_igemm_f16_t64x64 : K_igemm_f32_t64x64, kTile64.bn, kTile64.bm);
  if (far) return set(f16 ? K_igemm_f16_far128x128 : K_igemm_f32_far128x128, kFarTile, kFarTile);
  const int64_t row_bytes = a.K * es;
  const int64_t tiles32 = (int64_t)cdiv(a.M, kDirectTile) * cdiv(a.N, kDirectTile) * batch;
  if (persistent) {
    // One tile shape for the latency-oriented work, a larger one for heavy contractions.
    const double flops = 2.0 * a.M * a.N * a.K * (double)batch;
    const int64_t tiles = (int64_t)cdiv(a.M, kTile128x64.bm) * cdiv(a.N, kTile128x64.bn) * batch;
    if (tiles >= kTiledMinTiles && flops >= kTiledMinFlopsPersistent)
      return set(f16 ? K_igemm_f16_t128x64 : K_igemm_f32_t128x64, kTile128x64.bn, kTile128x64.bm);
    return set(f16 ? K_igemm_f16_direct4 : K_igemm_f32_direct4, kDirectTile, kDirectTile);
  }
  if (row_bytes < kQuadMinRowBytes && tiles32 < kDirectMaxTiles32) {
    // A wavefront walks a step or two of K: operands go to the matrix cores as they are loaded.
    if (tiles32 <= kSmallTileMaxTiles32) return set(f16 ? K_igemm_f16_direct4s : K_igemm_f32_direct4s, kSmallTile, kSmallTile);
    return set(f16 ? K_igemm_f16_direct4 : K_igemm_f32_direct4, kDirectTile, kDirectTile);
  }
  set(kTileKernels[0].ids[f16], kTileKernels[0].bn, kTileKernels[0].bm);
  KernelPlan *one = out;
  choose_tiles(&one, 1, false);
  return OPARA_OK;
}

int plan_pool(const opara_op_desc &op, const void *const *in, KernelPlan *out) {
  const opara_op_params &p = op.params;
  const bool f16 = op.dtype == OPARA_F16;
  const int ve = f16 ? 8 : 4;
  if (op.n_inputs != 1) return fail("pooling takes one input", op);
  if (p.h_in <= 0 || p.w_in <= 0 || p.c_in <= 0 || p.kh <= 0 || p.kw <= 0 || p.sh <= 0 || p.sw <= 0 ||
      p.ph < 0 || p.pw < 0 || p.ph >= p.kh || p.pw >= p.kw)
    return fail("bad pooling geometry", op);
  if (p.h_out != (p.h_in + 2 * p.ph - p.kh) / p.sh + 1 || p.w_out != (p.w_in + 2 * p.pw - p.kw) / p.sw + 1 ||
      p.h_out <= 0 || p.w_out <= 0)
    return fail("pooling output size does not match floor((in + 2*pad - k)/stride) + 1", op);
  PoolArgs a;
  std::memset(&a, 0, sizeof a);
  a.x = in[0]; a.y = op.out;
  a.H = p.h_in; a.W = p.w_in; a.C = p.c_in; a.Ho = p.h_out; a.Wo = p.w_out;
  a.kh = p.kh; a.kw = p.kw; a.sh = p.sh; a.sw = p.sw; a.ph = p.ph; a.pw = p.pw;
  a.is_avg = op.op_type == OPARA_AVGPOOL;
  if (p.batch < 0 || p.batch > 4096) return fail("bad image batch", op);
  a.B = p.batch > 0 ? p.batch : 1;
  const bool vec = (p.c_in % ve == 0) && aligned16(a.x) && aligned16(a.y);
  out->kernel = f16 ? (vec ? K_pool_f16_vec : K_pool_f16_scalar) : (vec ? K_pool_f32_vec : K_pool_f32_scalar);
  const int32_t chunks = vec ? p.c_in / ve : p.c_in;
  const int64_t items = (int64_t)a.B * p.h_out * p.w_out * chunks;
  const int64_t es = f16 ? 2 : 4, reach = (int64_t)1 << 31;
  const bool small = (int64_t)a.B * p.h_in * p.w_in * p.c_in * es < reach && (int64_t)a.B * p.h_out * p.w_out * p.c_in * es < reach;
  a.items = small ? (uint32_t)items : 0;
  a.div_cch = div_magic(chunks); a.div_Wo = div_magic(p.w_out); a.div_HoWo = div_magic(small ? p.h_out * p.w_out : 1);
  out->gx = cdiv(items, 256); out->gy = out->gz = 1; out->block = 256;
  out->args.pool = a;
  return OPARA_OK;
}

int plan_gap(const opara_op_desc &op, const void *const *in, KernelPlan *out) {
  const opara_op_params &p = op.params;
  if (op.n_inputs != 1 || p.h_in <= 0 || p.w_in <= 0 || p.c_in <= 0) return fail("bad global pooling shape", op);
  GapArgs a;
  std::memset(&a, 0, sizeof a);
  a.x = in[0]; a.y = op.out; a.HW = p.h_in * p.w_in; a.C = p.c_in;
  const int ve = op.dtype == OPARA_F16 ? 8 : 4;
  out->kernel = op.dtype == OPARA_F16 ? K_gap_f16 : K_gap_f32;
  if (p.batch < 0 || p.batch > 4096) return fail("bad image batch", op);
  // The vector form spreads the pixels of two chunks over a workgroup; with few pixels its
  // reductions cost more than the loads they save (7 x 7: 2.8 us against 2.3 us).
  a.vec = p.c_in % ve == 0 && aligned16(a.x) && aligned16(a.y) && a.HW >= kGapVecMinPixels;
  out->gx = cdiv(p.c_in, a.vec ? ve << kGapShare : 64); out->gy = p.batch > 0 ? p.batch : 1; out->gz = 1; out->block = 256;
  out->args.gap = a;
  return OPARA_OK;
}

int plan_row(const opara_op_desc &op, const void *const *in, KernelPlan *out) {
  const opara_op_params &p = op.params;
  const bool f16 = op.dtype == OPARA_F16;
  const int ve = f16 ? 8 : 4;
  if (p.m <= 0 || p.n <= 0) return fail("bad row-wise shape", op);
  RowArgs a;
  std::memset(&a, 0, sizeof a);
  a.y = op.out; a.n_in = op.n_inputs; a.rows = p.m; a.cols = p.n; a.eps = p.eps;
  bool vec = (p.n % ve == 0) && aligned16(a.y);
  for (int i = 0; i < op.n_inputs; ++i) { a.in[i] = in[i]; vec = vec && aligned16(in[i]); }
  const bool ln = op.op_type == OPARA_LAYERNORM;
  int variant;  // 0 wave, 1 block, 2 generic
  if (vec && p.n <= kRowGroupWave * ve * 2) variant = 0;
  else if (vec && p.n <= kRowGroupBlock * ve * kRowCacheChunks) variant = 1;
  else variant = 2;
  static const int ids[2][2][3] = {
      {{K_softmax_f32_wave, K_softmax_f32_block, K_softmax_f32_generic},
       {K_softmax_f16_wave, K_softmax_f16_block, K_softmax_f16_generic}},
      {{K_layernorm_f32_wave, K_layernorm_f32_block, K_layernorm_f32_generic},
       {K_layernorm_f16_wave, K_layernorm_f16_block, K_layernorm_f16_generic}}};
  out->kernel = ids[ln][f16][variant];
  out->block = 256;
  out->gx = variant == 0 ? cdiv(p.m, 256 / kRowGroupWave) : (uint32_t)p.m;
  out->gy = out->gz = 1;
  out->args.row = a;
  return OPARA_OK;
}

int plan_elt(const opara_op_desc &op, const void *const *in, KernelPlan *out) {
  const opara_op_params &p = op.params;
  const bool f16 = op.dtype == OPARA_F16;
  const int ve = f16 ? 8 : 4;
  if (p.m <= 0 || p.n <= 0) return fail("bad element-wise shape", op);
  EltArgs a;
  std::memset(&a, 0, sizeof a);
  a.y = op.out; a.n_in = op.n_inputs; a.n = (int64_t)p.m * p.n;
  a.op = op.op_type == OPARA_ADD ? 0 : op.op_type == OPARA_RELU ? 1 : 2;
  bool vec = (a.n % ve == 0) && aligned16(a.y);
  for (int i = 0; i < op.n_inputs; ++i) { a.in[i] = in[i]; vec = vec && aligned16(in[i]); }
  out->kernel = f16 ? (vec ? K_elt_f16_vec : K_elt_f16_scalar) : (vec ? K_elt_f32_vec : K_elt_f32_scalar);
  out->gx = cdiv(vec ? a.n / ve : a.n, 256); out->gy = out->gz = 1; out->block = 256;
  out->args.elt = a;
  return OPARA_OK;
}

int plan_concat(const opara_op_desc &op, const void *const *in, KernelPlan *out) {
  const opara_op_params &p = op.params;
  const bool f16 = op.dtype == OPARA_F16;
  const int ve = f16 ? 8 : 4;
  if (p.m <= 0) return fail("bad concat shape", op);
  ConcatArgs a;
  std::memset(&a, 0, sizeof a);
  a.y = op.out; a.n_in = op.n_inputs; a.rows = p.m;
  bool vec = aligned16(a.y);
  int32_t off = 0, widest = 0;
  for (int i = 0; i < op.n_inputs; ++i) {
    if (p.in_cols[i] <= 0) return fail("concat input with no columns", op);
    a.in[i] = in[i]; a.cols[i] = p.in_cols[i]; a.col_off[i] = off;
    off += p.in_cols[i];
    if (p.in_cols[i] > widest) widest = p.in_cols[i];
    vec = vec && (p.in_cols[i] % ve == 0) && aligned16(in[i]);
  }
  for (int i = 0; i < op.n_inputs; ++i) a.div_cols[i] = div_magic(vec ? a.cols[i] / ve : a.cols[i]);
  if (p.n != off) return fail("concat: n must equal the sum of in_cols", op);
  a.out_cols = off;
  out->kernel = f16 ? (vec ? K_concat_f16_vec : K_concat_f16_scalar) : (vec ? K_concat_f32_vec : K_concat_f32_scalar);
  out->gx = cdiv((int64_t)p.m * (vec ? widest / ve : widest), 256);
  out->gy = (uint32_t)op.n_inputs; out->gz = 1; out->block = 256;
  out->args.concat = a;
  return OPARA_OK;
}

}  // namespace

// Tile shapes of contractions that run together: those of a wave that becomes a group kernel
// (`grouped`, also where there is only one beside operators of other types), or a launch of its own.
// Small tiles finish one operator sooner (more CUs share it), large ones move
// fewer bytes per multiply-add; what counts is the longer of the time the work takes on all
// CUs together and the time the longest workgroup takes.  For every bound on the latter,
// each operator takes its cheapest tile shape within it; the best bound wins.  The bounds are
// visited in increasing order, and each only changes the one operator whose shape it admits
// (trying every operator again under every bound took seconds for a wave of some thousand).
void choose_tiles(KernelPlan *const *plans, int n, bool grouped) {
  struct Option { double longest, work; int op, shape; };
  std::vector<Option> options;
  for (int i = 0; i < n; ++i) {
    const IgemmArgs &a = plans[i]->args.igemm;
    const bool f16 = tile_kernel_is_f16(plans[i]->kernel);
    const double steps = std::ceil(a.K * (f16 ? 2.0 : 4.0) / 128.0);
    for (int k = 0; k < kTileKernelCount; ++k) {
      const TileKernel &t = kTileKernels[k];
      const double tiles = (double)cdiv(a.M, t.bm) * cdiv(a.N, t.bn) * plans[i]->gz;
      const double least = f16 ? 0.0 : t.bn * t.bm * 32 * 2.0 / 0.6e6;
      Option o;
      o.op = i;
      o.shape = k;
      o.longest = steps * std::max(t.alone, least) + t.fixed;
      o.work = tiles * (steps * std::max(t.busy, least) + t.fixed) / kCus * (grouped ? t.together : 1.0);
      if (!grouped && tiles > kCus && tiles < 4 * kCus)      // a single launch: whole rounds over the CUs
        o.work *= std::ceil(tiles / kCus) * kCus / tiles;
      options.push_back(o);
    }
  }
  std::sort(options.begin(), options.end(), [](const Option &a, const Option &b) {
    return std::tie(a.longest, a.op, a.shape) < std::tie(b.longest, b.op, b.shape);
  });
  // take[i]: the operator's cheapest shape so far, and how many of these decisions (in the order
  // they fall) belong to the best bound.
  std::vector<const Option *> take(n, nullptr);
  std::vector<const Option *> made;
  double work = 0.0, longest = 0.0, best = -1.0;
  size_t best_made = 0;
  int missing = n;
  for (size_t j = 0; j < options.size(); ++j) {
    const Option &o = options[j];
    const Option *&t = take[o.op];
    if (!t || o.work < t->work) {
      work += o.work - (t ? t->work : 0.0);
      missing -= t ? 0 : 1;
      t = &o;
      longest = o.longest;                                 // no operator had a longer one
      made.push_back(&o);
    }
    if (missing || (j + 1 < options.size() && options[j + 1].longest == o.longest)) continue;
    const double cost = std::max(work, longest);
    if (best < 0.0 || cost < best) { best = cost; best_made = made.size(); }
  }
  std::vector<int> pick(n, 0);
  for (size_t j = 0; j < best_made; ++j) pick[made[j]->op] = made[j]->shape;
  for (int i = 0; i < n; ++i) {
    const TileKernel &t = kTileKernels[pick[i]];
    const IgemmArgs &a = plans[i]->args.igemm;
    plans[i]->kernel = t.ids[tile_kernel_is_f16(plans[i]->kernel)];
    plans[i]->gx = cdiv(a.M, t.bm);
    plans[i]->gy = cdiv(a.N, t.bn);
    plans[i]->args.igemm.div_gx = div_magic((int64_t)plans[i]->gx);
  }
}

int tail_kernel(int kernel_id) {
  switch (kernel_id) {
#define TAIL(name) case K_igemm_f16_##name: return K_igemm_f16_##name##_tail; case K_igemm_f32_##name: return K_igemm_f32_##name##_tail;
    TAIL(quad4s) TAIL(quad4) TAIL(quad64x4) TAIL(quad64x64) TAIL(tile64x64) TAIL(t128x64) TAIL(tile128x128)
#undef TAIL
    default: return -1;
  }
}

bool tile_choice_open(int kernel_id) {
  return std::any_of(kTileKernels, kTileKernels + kTileKernelCount,
                     [&](const TileKernel &t) { return t.ids[0] == kernel_id || t.ids[1] == kernel_id; });
}

int plan_op(const opara_op_desc &op, const void *const *in, int kind, KernelPlan *out) {
  std::memset(out, 0, sizeof *out);
  int rc;
  switch (op.op_type) {
    case OPARA_CONV2D: case OPARA_GEMM: case OPARA_BGEMM: rc = plan_igemm(op, in, kind, out); break;
    case OPARA_MAXPOOL: case OPARA_AVGPOOL: rc = plan_pool(op, in, out); break;
    case OPARA_GAVGPOOL: rc = plan_gap(op, in, out); break;
    case OPARA_LAYERNORM: case OPARA_SOFTMAX: rc = plan_row(op, in, out); break;
    case OPARA_GELU: case OPARA_RELU: case OPARA_ADD: rc = plan_elt(op, in, out); break;
    case OPARA_CONCAT: rc = plan_concat(op, in, out); break;
    default: set_error("unknown operator type %d", op.op_type); return OPARA_EINVAL;
  }
  if (rc != OPARA_OK) return rc;
  if (out->gx == 0 || out->gy == 0 || out->gz == 0 || out->gy > 65535u || out->gz > 65535u) {
    set_error("operator type %d: launch grid out of range", op.op_type);
    return OPARA_EUNSUPPORTED;
  }
  return OPARA_OK;
}

}  // namespace opara
