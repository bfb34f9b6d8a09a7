// Attention of one head and sixteen query rows per workgroup (included by kernels.hip).
//
// Scores, softmax and context are three operators of the DAG; where they follow one another
// with nothing beside them, the fused executor runs them as this one kernel.  Every operator's
// result is still written, and each stage reads what the unmerged kernels would have read: the
// stored fp16 values of the stage before.
//
// What bounds it: three launches and two passes of the scores through memory, at these sizes
// (12 heads x 128 x 64: 1.6 MB in all, half of it scores and probabilities) hardly any arithmetic.  Sixteen rows per workgroup because
// a head has few rows (128: 96 workgroups, 512: 384); a row of up to kAttnMaxCols scores fits one
// 16-byte chunk per lane of a wavefront.  The columns are dealt to the four wavefronts in tiles;
// a wavefront stages its own tiles of K, and later of V, in its own ring and waits for its own
// loads only.  V is consumed transposed: ds_read_b64_tr_b16 hands every group of sixteen lanes a
// 4 x 16 block with the lane as column.
// Measured, fp16, 12 heads of 64 (scores + softmax + context as three launches -> one): 128 rows
// 11.6 -> 4.3 us, 512 rows 22.6 -> 12.3 us (an empty launch: 2.2).  At 512 rows the serial chain
// of one workgroup bounds it: loads, scores, softmax and context wait for one another.

// Four rows k .. k+3 of sixteen columns: lane i of a group of sixteen gives the address of the
// i % 4-th run of four columns of row k + i / 4 and receives column i of the four rows.
__device__ __forceinline__ half4 lds_read_transposed(const unsigned char *p) {
  typedef short s4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s4 *)(uintptr_t)lds_address(p)));
}
__device__ __forceinline__ void meet_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory"); }

constexpr int kAttnPitch = kAttnMaxCols * 2 + 16;          // bytes per row of probabilities in LDS
constexpr int kAttnRing = 4 * 2048;                        // bytes per wavefront: four tiles of K or two of V
constexpr int kLdsAttention = 16 * kAttnPitch + 4 * (2048 + kAttnRing);

template <typename AR>
__device__ __forceinline__ void attention_body(const AR &a, const Blk &b, unsigned char *lds) {
  typedef half_t T;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int grp = lane >> 4, r16 = lane & 15, l8 = lane >> 3, chunk = (lane & 7) ^ l8;
  int tile_x, z;
  xcd_tile(b, a.div_gx, tile_x, z);                                // row tiles of one head share an L2
  const int m0 = tile_x * 16;
  const int N = a.N;
  const i32x4 qbuf = buffer_of((const T *)a.q + (int64_t)z * a.q_bs, a.q_bytes);
  const i32x4 kbuf = buffer_of((const T *)a.k + (int64_t)z * a.k_bs, a.k_bytes);
  const i32x4 vbuf = buffer_of((const T *)a.v + (int64_t)z * a.v_bs, a.v_bytes);
  unsigned char *prob = lds;
  unsigned char *own = lds + 16 * kAttnPitch + wave * (2048 + kAttnRing);   // query rows, then the ring
  const uint32_t qlds = lds_address(own), ring = qlds + 2048;
  const unsigned char *rbase = own + 2048;

  // ---- scores: this wavefront's tiles of sixteen columns are wave, wave + 4, ...
  const int tiles = (N + 15) >> 4, mine = (tiles - wave + 3) >> 2;
  const bool kin = chunk * 8 < a.D;                         // inside a row of D halves
  auto load_rows = [&](const i32x4 &buf, int row, int rows, uint32_t ld, uint32_t at) {
    lds_load16(buf, kin && row < rows ? ((uint32_t)row * ld + (uint32_t)chunk * 8u) * 2u : kOperandMaxBytes, 0, at);
  };
  auto load_k = [&](int i) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      load_rows(kbuf, (wave + i * 4) * 16 + h * 8 + l8, N, (uint32_t)a.ldk, ring + (i & 3) * 2048 + h * 1024);
  };
  if (mine > 0)                                             // no load may outlive its wavefront
#pragma unroll
    for (int h = 0; h < 2; ++h) load_rows(qbuf, m0 + h * 8 + l8, a.M, (uint32_t)a.ldq, qlds + h * 1024);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i < mine) load_k(i);
  const int c0 = (grp ^ (r16 & 7)) * 16, c1 = ((4 + grp) ^ (r16 & 7)) * 16;   // this lane's two chunks of a row
  half8 qf[2];
#pragma nounroll
  for (int i = 0; i < mine; ++i) {
    if (i + 3 < mine) wait_loads<6>();
    else wait_loads<0>();
    if (i == 0) { qf[0] = *(const half8 *)(own + r16 * 128 + c0); qf[1] = *(const half8 *)(own + r16 * 128 + c1); }
    const unsigned char *row = rbase + (i & 3) * 2048 + r16 * 128;
    const half8 k0 = *(const half8 *)(row + c0), k1 = *(const half8 *)(row + c1);
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");    // the slot has been read: it may be refilled
    if (i + 4 < mine) load_k(i + 4);
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = mma16<T>(k0, qf[0], acc);
    acc = mma16<T>(k1, qf[1], acc);
    half4 s;
#pragma unroll
    for (int e = 0; e < 4; ++e) s[e] = (T)(acc[e] * a.alpha_s);
    *(half4 *)(prob + r16 * kAttnPitch + ((wave + i * 4) * 16 + grp * 4) * 2) = s;
  }

  // ---- V follows K into the ring, 32 rows a tile, while the softmax runs
  const int vtiles = (N + 31) >> 5, vmine = (vtiles - wave + 3) >> 2;
  const bool vin = chunk * 8 < a.D2;
  auto load_v = [&](int i) {
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int row = (wave + i * 4) * 32 + h * 8 + l8;
      lds_load16(vbuf, vin && row < N ? ((uint32_t)row * (uint32_t)a.ldv + (uint32_t)chunk * 8u) * 2u : kOperandMaxBytes, 0,
                 ring + (i & 1) * 4096 + h * 1024);
    }
  };
#pragma unroll
  for (int i = 0; i < 2; ++i)
    if (i < vmine) load_v(i);
  meet_lds();                                               // all columns of the sixteen rows are there

  // ---- softmax: four rows per wavefront; 16, 32 or 64 lanes share a row, eight columns each, so
  // that a wavefront takes four, two or one of them at a time
  const int share = N <= 128 ? 4 : N <= 256 ? 5 : 6;        // log2 of the lanes that share a row
  const int col = (lane & ((1 << share) - 1)) * 8;
  auto row_of = [&](int r) { return wave * 4 + (lane >> share) + (r << (6 - share)); };
  half8 sv[4], pv[4];
  auto softmax_rows = [&](auto lanes_tag) {                 // stage by stage: the rows' reductions overlap
    constexpr int LANES = decltype(lanes_tag)::value, ROWS = LANES / 16;
    float v[ROWS][8], mx[ROWS], sum[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      sv[r] = *(const half8 *)(prob + row_of(r) * kAttnPitch + col * 2);
      mx[r] = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[r][e] = (float)sv[r][e];
        mx[r] = fmaxf(mx[r], col + e < N ? v[r][e] : -INFINITY);
      }
    }
#pragma unroll
    for (int off = LANES / 2; off > 0; off >>= 1)
#pragma unroll
      for (int r = 0; r < ROWS; ++r) mx[r] = fmaxf(mx[r], __shfl_xor(mx[r], off, 64));
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      sum[r] = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[r][e] = col + e < N ? expf(v[r][e] - mx[r]) : 0.f;
        sum[r] += v[r][e];
      }
    }
#pragma unroll
    for (int off = LANES / 2; off > 0; off >>= 1)
#pragma unroll
      for (int r = 0; r < ROWS; ++r) sum[r] += __shfl_xor(sum[r], off, 64);
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
      const float inv = 1.0f / sum[r];
#pragma unroll
      for (int e = 0; e < 8; ++e) pv[r][e] = col + e < N ? (T)(v[r][e] * inv) : (T)0.f;
      *(half8 *)(prob + row_of(r) * kAttnPitch + col * 2) = pv[r];
    }
  };
  if (share == 4) softmax_rows(std::integral_constant<int, 16>{});
  else if (share == 5) softmax_rows(std::integral_constant<int, 32>{});
  else softmax_rows(std::integral_constant<int, 64>{});
  meet_lds();

  // ---- context: this wavefront's rows of V, all columns; partial sums meet below
  floatx4 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma nounroll
  for (int i = 0; i < vmine; ++i) {
    if (i + 1 < vmine) wait_loads<4>();
    else wait_loads<0>();
    const half8 pf = *(const half8 *)(prob + r16 * kAttnPitch + ((wave + i * 4) * 32 + grp * 8) * 2);
    const unsigned char *tile = rbase + (i & 1) * 4096;
    half4 vf[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int row = grp * 8 + h * 4 + (r16 >> 2);
        vf[j][h] = lds_read_transposed(tile + row * 128 + (((j * 2 + ((r16 >> 1) & 1)) ^ (row & 7)) * 16) + (r16 & 1) * 8);
      }
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
    if (i + 2 < vmine) load_v(i + 2);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const half8 af = __builtin_shufflevector(vf[j][0], vf[j][1], 0, 1, 2, 3, 4, 5, 6, 7);
      acc[j] = mma16<T>(af, pf, acc[j]);
    }
  }

  // ---- results: scores and probabilities from registers, context from the partial sums
  auto store_row = [&](void *base, int r, half8 v) {
    typedef half8 VU __attribute__((aligned(2)));
    const int m = m0 + row_of(r);
    if (m >= a.M || col >= N) return;
    T *dst = (T *)base + ((int64_t)z * a.M + m) * N + col;
    if (col + 7 < N) {
      *(VU *)dst = v;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (col + e < N) dst[e] = v[e];
    }
  };
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (r < 1 << (share - 4)) { store_row(a.s, r, sv[r]); store_row(a.p, r, pv[r]); }
  constexpr int PITCH = 68;                                 // floats per row of a partial tile
  float *part = (float *)(own + 2048);
#pragma unroll
  for (int j = 0; j < 4; ++j) *(floatx4 *)(part + r16 * PITCH + j * 16 + grp * 4) = acc[j];
  meet_lds();
  const int pm = t >> 4, pn = (t & 15) * 4;
  if (m0 + pm < a.M && pn < a.D2) {
    const unsigned char *at = lds + 16 * kAttnPitch + 2048 + (pm * PITCH + pn) * 4;
    floatx4 sum = *(const floatx4 *)at;
#pragma unroll
    for (int q = 1; q < 4; ++q) sum += *(const floatx4 *)(at + q * (2048 + kAttnRing));
    half4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = (T)(sum[e] * a.alpha_c);
    typedef half4 QU __attribute__((aligned(2)));
    *(QU *)((T *)a.y + (int64_t)z * a.y_bs + (int64_t)(m0 + pm) * a.ldy + pn) = o;
  }
}
