// Operators that share a kernel in the fused executor (host only, no HIP calls).
//
// A node of the executor's chain costs 1.7 us (an empty kernel) to 2.3 us (a small operator), so a
// wave whose only operator consumes the only operator of the wave before is worth no launch of its
// own when the producer's kernel can go on to compute it.  Every operator's result is still
// written, and the consumer computes from the stored (rounded) values: element-wise tails and
// concatenations written in place are the same bits; attention adds its sums in another order than
// the three kernels do (softmax over the lanes of a row, context over four wavefronts) and agrees
// to rounding.
//
// An operator that is alone in its wave runs when everything of earlier waves is complete,
// and the operators of a merge are alone in theirs: whatever else they read is ready when the
// first of them starts.  Buffers must not overlap (a caller may have let the result of a later
// operator replace what an earlier one reads); merges with overlapping buffers are not made.
#include <algorithm>
#include <cstring>
#include "opara_internal.h"

namespace opara {
namespace {

struct Range { uintptr_t begin, end; };
Range range_of(const void *p, int64_t bytes) { return {(uintptr_t)p, (uintptr_t)p + (uintptr_t)bytes}; }
bool disjoint(const Range &a, const Range &b) { return a.end <= b.begin || b.end <= a.begin; }
bool disjoint(const Range &a, std::initializer_list<Range> l) {
  return std::all_of(l.begin(), l.end(), [&](const Range &b) { return disjoint(a, b); });
}
bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }
bool vectors(const void *p, int64_t ld, int64_t bs) { return aligned16(p) && ld % 8 == 0 && bs % 8 == 0; }

// scores (batched product) -> softmax -> context (batched product with a [K][N] operand).
bool merge_attention(const opara_dag *g, int32_t u, int32_t v, int32_t w, Merge *out) {
  const opara_op_desc &du = g->ops[u], &dv = g->ops[v], &dw = g->ops[w];
  if (du.op_type != OPARA_BGEMM || dv.op_type != OPARA_SOFTMAX || dw.op_type != OPARA_BGEMM) return false;
  if (du.dtype != OPARA_F16 || dv.dtype != OPARA_F16 || dw.dtype != OPARA_F16) return false;
  if (dv.n_inputs != 1 || dv.inputs[0] != u || dw.inputs[0] != v || dw.inputs[1] == u || dw.inputs[1] == v) return false;
  const IgemmArgs &s = g->plan[u].args.igemm, &c = g->plan[w].args.igemm;
  const RowArgs &r = g->plan[v].args.row;
  const int64_t heads = g->plan[u].gz, rows = heads * s.M, cells = (int64_t)s.M * s.N;
  if (s.b_kmajor || s.relu || s.bias || !c.b_kmajor || c.relu || c.bias) return false;
  if (s.K > kAttnMaxWidth || s.K % 8 || s.N > kAttnMaxCols || c.N > kAttnMaxWidth || c.N % 8) return false;
  if (!vectors(s.x, s.lda, s.a_bs) || !vectors(s.w, s.ldb, s.b_bs) || !vectors(c.w, c.ldb, c.b_bs)) return false;
  if (s.ldy != s.N || s.y_bs != cells || r.in[0] != s.y || r.rows != rows || r.cols != s.N) return false;
  if (c.x != r.y || (int64_t)g->plan[w].gz != heads || c.M != s.M || c.K != s.N || c.lda != s.N || c.a_bs != cells) return false;
  const int64_t q_bytes = 2 * ((int64_t)(s.M - 1) * s.lda + s.K), k_bytes = 2 * ((int64_t)(s.N - 1) * s.ldb + s.K),
                v_bytes = 2 * ((int64_t)(c.K - 1) * c.ldb + c.N);
  if (std::max({q_bytes, k_bytes, v_bytes}) >= (int64_t)kOperandMaxBytes) return false;
  const Range q = range_of(s.x, 2 * (heads - 1) * s.a_bs + q_bytes), k = range_of(s.w, 2 * (heads - 1) * s.b_bs + k_bytes),
              vv = range_of(c.w, 2 * (heads - 1) * c.b_bs + v_bytes), sc = range_of(s.y, 2 * heads * cells),
              pr = range_of(r.y, 2 * heads * cells),
              y = range_of(c.y, 2 * ((heads - 1) * c.y_bs + (int64_t)(c.M - 1) * c.ldy + c.N));
  if (!disjoint(sc, vv) || !disjoint(pr, {q, k, vv, sc}) || !disjoint(y, {q, k, vv, sc, pr})) return false;
  out->count = 3;
  out->ops[0] = u; out->ops[1] = v; out->ops[2] = w;
  KernelPlan &p = out->plan;
  std::memset(&p, 0, sizeof p);
  p.kernel = K_attention_f16;
  p.gx = (uint32_t)((s.M + 15) / 16); p.gy = (uint32_t)heads; p.gz = 1; p.block = 256; p.tag = u;
  AttnArgs &a = p.args.attn;
  a.q = s.x; a.k = s.w; a.v = c.w; a.s = s.y; a.p = r.y; a.y = c.y;
  a.q_bs = s.a_bs; a.k_bs = s.b_bs; a.v_bs = c.b_bs; a.y_bs = c.y_bs; a.ldy = c.ldy;
  a.ldq = (int32_t)s.lda; a.ldk = (int32_t)s.ldb; a.ldv = (int32_t)c.ldb;
  a.M = s.M; a.N = s.N; a.D = s.K; a.D2 = c.N;
  a.q_bytes = (uint32_t)q_bytes; a.k_bytes = (uint32_t)k_bytes; a.v_bytes = (uint32_t)v_bytes;
  a.div_gx = div_magic(p.gx);
  a.alpha_s = s.alpha; a.alpha_c = c.alpha;
  return true;
}

// contraction -> element-wise operator of its size, in whole vectors.  The contractions fed
// through workgroup memory have a form with such a tail.
bool merge_tail(const opara_dag *g, int32_t u, int32_t v, Merge *out) {
  const opara_op_desc &du = g->ops[u], &dv = g->ops[v];
  const KernelPlan &pu = g->plan[u];
  if (du.op_type != OPARA_CONV2D && du.op_type != OPARA_GEMM) return false;
  if (dv.op_type != OPARA_ADD && dv.op_type != OPARA_RELU && dv.op_type != OPARA_GELU) return false;
  if (du.dtype != dv.dtype || tail_kernel(pu.kernel) < 0) return false;
  const IgemmArgs &c = pu.args.igemm;
  const EltArgs &e = g->plan[v].args.elt;
  const int64_t es = du.dtype == OPARA_F16 ? 2 : 4, cells = (int64_t)c.M * c.N;
  if (c.ldy != c.N || e.n != cells || e.n_in > 3) return false;
  if (c.N % 4 || es * cells >= (int64_t)1 << 31 || !aligned16(e.y)) return false;
  TailArgs t;
  std::memset(&t, 0, sizeof t);
  t.y = e.y; t.n_in = e.n_in; t.op = e.op; t.self = -1;
  const Range y = range_of(c.y, es * cells), ty = range_of(e.y, es * cells),
              x = range_of(c.x, c.x_bytes), w = range_of(c.w, c.w_bytes), bias = range_of(c.bias, c.bias ? 4 * (int64_t)c.N : 0);
  if (!disjoint(ty, {y, x, w, bias})) return false;
  for (int q = 0; q < c.n_extra; ++q)
    if (!disjoint(ty, range_of(c.extra[q], es * cells))) return false;
  int others = 0;
  for (int q = 0; q < e.n_in; ++q) {
    if (dv.inputs[q] == u) {
      if (t.self >= 0 || e.in[q] != c.y) return false;
      t.self = q;
      continue;
    }
    if (others == 2 || !aligned16(e.in[q])) return false;
    const Range r = range_of(e.in[q], es * cells);
    if (!disjoint(r, {y, ty})) return false;
    t.in[others++] = e.in[q];
  }
  if (t.self < 0) return false;
  out->count = 2;
  out->ops[0] = u; out->ops[1] = v;
  out->plan = pu;
  out->plan.kernel = tail_kernel(pu.kernel);
  out->plan.tail = t;
  return true;
}

}  // namespace

namespace {
std::vector<std::vector<int32_t>> waves_of(const opara_dag *g) {
  std::vector<int32_t> wave(g->n, 0);
  std::vector<std::vector<int32_t>> waves;
  for (int32_t i = 0; i < g->n; ++i) {
    const int32_t v = g->topo[i];
    for (int32_t j = g->pred_off[v]; j < g->pred_off[v + 1]; ++j) wave[v] = std::max(wave[v], wave[g->pred[j]] + 1);
    if (wave[v] >= (int32_t)waves.size()) waves.resize(wave[v] + 1);
    waves[wave[v]].push_back(v);
  }
  return waves;
}

// Everything an operator reads or writes.
std::vector<Range> touched(const opara_dag *g, int32_t v) {
  const opara_op_desc &d = g->ops[v];
  const KernelPlan &p = g->plan[v];
  const int64_t es = d.dtype == OPARA_F16 ? 2 : 4;
  std::vector<Range> r;
  auto add = [&](const void *q, int64_t elements) { if (q) r.push_back(range_of(q, es * elements)); };
  switch (d.op_type) {
    case OPARA_CONV2D: case OPARA_GEMM: case OPARA_BGEMM: {
      const IgemmArgs &a = p.args.igemm;
      const int64_t z = p.gz - 1;
      add(a.x, a.gather ? (int64_t)(a.M / a.HoWo) * a.img_stride : z * a.a_bs + (int64_t)(a.M - 1) * a.lda + a.K);
      add(a.w, z * a.b_bs + (int64_t)((a.b_kmajor ? a.K : a.N) - 1) * a.ldb + (a.b_kmajor ? a.N : a.K));
      add(a.y, z * a.y_bs + (int64_t)(a.M - 1) * a.ldy + a.N);
      for (int q = 0; q < a.n_extra; ++q) add(a.extra[q], (int64_t)a.M * a.N);
      if (a.bias) r.push_back(range_of(a.bias, 4 * (int64_t)a.N));
      break;
    }
    case OPARA_MAXPOOL: case OPARA_AVGPOOL:
      add(p.args.pool.x, (int64_t)p.args.pool.B * p.args.pool.H * p.args.pool.W * p.args.pool.C);
      add(p.args.pool.y, (int64_t)p.args.pool.B * p.args.pool.Ho * p.args.pool.Wo * p.args.pool.C);
      break;
    case OPARA_GAVGPOOL:
      add(p.args.gap.x, (int64_t)p.gy * p.args.gap.HW * p.args.gap.C);
      add(p.args.gap.y, (int64_t)p.gy * p.args.gap.C);
      break;
    case OPARA_LAYERNORM: case OPARA_SOFTMAX:
      for (int q = 0; q < p.args.row.n_in; ++q) add(p.args.row.in[q], (int64_t)p.args.row.rows * p.args.row.cols);
      add(p.args.row.y, (int64_t)p.args.row.rows * p.args.row.cols);
      break;
    case OPARA_CONCAT:
      for (int q = 0; q < p.args.concat.n_in; ++q) add(p.args.concat.in[q], (int64_t)p.args.concat.rows * p.args.concat.cols[q]);
      add(p.args.concat.y, (int64_t)p.args.concat.rows * p.args.concat.out_cols);
      break;
    default:
      for (int q = 0; q < p.args.elt.n_in; ++q) add(p.args.elt.in[q], p.args.elt.n);
      add(p.args.elt.y, p.args.elt.n);
  }
  return r;
}
}  // namespace

// A concatenation that makes up its wave and joins results of element-wise operators: each of them
// writes its result twice, and the concatenation needs no launch (one of four per cell of
// the NASNet-like network: 101 -> 90 us).  Nothing that runs from the first of them on
// may touch the concatenation's buffer.
std::vector<ConcatMerge> find_concat_merges(const opara_dag *g, const std::vector<Merge> &taken) {
  std::vector<char> used(g->n, 0);
  for (const Merge &m : taken)
    for (int32_t i = 0; i < m.count; ++i) used[m.ops[i]] = 1;
  const std::vector<std::vector<int32_t>> waves = waves_of(g);
  std::vector<size_t> wave(g->n);
  for (size_t w = 0; w < waves.size(); ++w)
    for (int32_t v : waves[w]) wave[v] = w;
  std::vector<ConcatMerge> found;
  for (size_t w = 1; w < waves.size(); ++w) {
    const int32_t v = waves[w][0];
    if (waves[w].size() != 1 || used[v] || g->ops[v].op_type != OPARA_CONCAT) continue;
    const bool f16 = g->ops[v].dtype == OPARA_F16;
    if (g->plan[v].kernel != (f16 ? K_concat_f16_vec : K_concat_f32_vec)) continue;
    const ConcatArgs &c = g->plan[v].args.concat;
    const Range y = range_of(c.y, (f16 ? 2 : 4) * (int64_t)c.rows * c.out_cols);
    ConcatMerge m;
    m.concat = v;
    size_t first = w;                               // wave of the first part
    bool ok = true;
    for (int q = 0; q < c.n_in && ok; ++q) {
      const int32_t u = g->ops[v].inputs[q];
      ok = u >= 0 && !used[u] && std::count(m.ops.begin(), m.ops.end(), u) == 0 && g->plan[u].kernel == (f16 ? K_elt_f16_vec : K_elt_f32_vec);
      if (!ok) break;
      EltArgs e = g->plan[u].args.elt;
      const int ve = f16 ? 8 : 4;
      ok = e.n == (int64_t)c.rows * c.cols[q] && e.y == c.in[q] && e.n / ve < (int64_t)1 << 31;
      e.also = (unsigned char *)c.y + (f16 ? 2 : 4) * (int64_t)c.col_off[q];
      e.also_cols = c.cols[q];
      e.also_pitch = c.out_cols;
      e.div_also = div_magic(c.cols[q] / ve);
      first = std::min(first, wave[u]);
      m.ops.push_back(u);
      m.args.push_back(e);
    }
    for (size_t i = first; i < w && ok; ++i)
      for (int32_t u : waves[i])
        for (const Range &r : touched(g, u)) ok = ok && disjoint(y, r);
    if (!ok) continue;
    for (int32_t u : m.ops) used[u] = 1;
    found.push_back(m);
  }
  return found;
}

std::vector<Merge> find_merges(const opara_dag *g) {
  const std::vector<std::vector<int32_t>> waves = waves_of(g);
  std::vector<int32_t> alone;                       // the only operator of a wave, -1 if there are more
  for (const auto &w : waves) alone.push_back(w.size() == 1 ? w[0] : -1);
  std::vector<Merge> found;
  for (size_t w = 0; w + 1 < waves.size(); ++w) {
    Merge m;
    if (alone[w] < 0 || alone[w + 1] < 0) continue;
    if (w + 2 < waves.size() && alone[w + 2] >= 0 && merge_attention(g, alone[w], alone[w + 1], alone[w + 2], &m)) {
      found.push_back(m);
      w += (size_t)m.count - 1;
    } else if (merge_tail(g, alone[w], alone[w + 1], &m)) {
      found.push_back(m);
      ++w;
    }
  }
  return found;
}

}  // namespace opara
