// Operator kernels for gfx950 (CDNA4) and their launcher.
//
// The paper runs vendor-library kernels (Sec. 5.1); these are this library's own.
// Dense contractions (convolution as implicit GEMM, GEMM, batched GEMM) use the
// matrix cores; everything else is a coalesced 16-byte-per-lane streaming kernel
// with wavefront (64-lane) reductions where rows are reduced.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <algorithm>
#include <type_traits>
#include "kernel_args.h"
#include "launch.h"

namespace opara {

typedef _Float16 half_t;
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Position of a workgroup in its operator's launch grid.  An ordinary launch fills it from
// blockIdx and the launch's arguments; the persistent executor hands out grid positions itself.
struct Blk {
  int x, y, z, gx, gy;
  int lin;                                 // y * gx + x
  bool remap;                              // apply the XCD-aware tile remap (hardware launch order only)
};
__device__ __forceinline__ Blk launch_blk(const LaunchArgs &l) {
  return Blk{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, l.gx, l.gy, (int)blockIdx.y * l.gx + (int)blockIdx.x, true};
}
// floor(n / d) with m = min(2^32 / d, 2^32 - 1): the product underestimates by at most one.
__device__ __forceinline__ uint32_t fast_div(uint32_t n, uint32_t d, uint32_t m) {
  const uint32_t q = __umulhi(n, m);
  return n - q * d >= d ? q + 1 : q;
}

template <typename T> struct Vec16;
template <> struct Vec16<half_t> { typedef half8 type; typedef half4 quad; static constexpr int N = 8; };
template <> struct Vec16<float> { typedef floatx4 type; typedef floatx4 quad; static constexpr int N = 4; };
template <typename T> struct VecRun { static constexpr int N = 16 / (4 * sizeof(T)); };   // runs of four elements in 16 bytes

// Access policy of a body.  Ordinary launches use plain loads and stores: kernel
// boundaries make results visible.  Inside the persistent and chained executors an
// operator's inputs were written by other workgroups of the same launch, possibly on another
// XCD with its own L2; there results are stored with agent-scope (device-coherent) accesses,
// which the hardware completes at the point all XCDs share, so that a completion counter
// published after a wait for the stores is all the synchronisation a consumer needs: no cache
// write-back.  Loads stay plain and follow a cache invalidate.
constexpr int kCohStore = 1;

template <typename V, typename P> __device__ __forceinline__ V ldg(const P *p) { return *(const V *)p; }

template <bool COH, typename V, typename P>
__device__ __forceinline__ void stg(P *p, const V &v) {
  if constexpr (!COH) {
    *(V *)p = v;
  } else if constexpr (sizeof(V) == 16) {
    // One 16-byte write-through store (what a relaxed agent-scope atomic store compiles to for
    // 8 bytes, `global_store_dwordx2 ... sc1`, in its four-dword form): the language has no
    // 16-byte atomic, and two 8-byte ones reach memory as two partial-line writes.  Like any plain
    // store of the machine it takes element alignment.  The nop
    // covers the wait state a store of more than 8 bytes needs before its data registers
    // may be overwritten.
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 q = __builtin_bit_cast(u32x4, v);
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(p), "v"(q) : "memory");
  } else if constexpr (sizeof(V) == 8) {
    uint64_t q;
    __builtin_memcpy(&q, &v, 8);
    __hip_atomic_store((uint64_t *)p, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else if constexpr (sizeof(V) == 4) {
    uint32_t q;
    __builtin_memcpy(&q, &v, 4);
    __hip_atomic_store((uint32_t *)p, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    static_assert(sizeof(V) == 2, "access width");
    uint16_t q;
    __builtin_memcpy(&q, &v, 2);
    __hip_atomic_store((uint16_t *)p, q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// ---------------------------------------------------------------------------------
// Implicit GEMM on the matrix cores.
//
// Workgroup tile: BN output columns (channels) x BM output rows (pixels); K is walked
// in slices of 64 bytes per row (32 halves / 16 floats).  Both operands are staged in
// LDS with K fastest and an 80-byte row pitch, so that the 16-byte fragment reads of
// 16 consecutive rows fall into distinct banks.  Weights feed the MFMA "A" side and
// pixels the "B" side: each lane then owns four consecutive output channels of one
// pixel, which is a contiguous 8/16-byte store in the [row][channel] output.
// The mapping of K positions onto MFMA K slots is the same for both operands, which is
// all a dot product needs, so the same 16-byte fragment load serves fp16 and fp32.
// ---------------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ floatx4 mma16(typename Vec16<T>::type a, typename Vec16<T>::type b, floatx4 c);
template <> __device__ __forceinline__ floatx4 mma16<half_t>(half8 a, half8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}
template <> __device__ __forceinline__ floatx4 mma16<float>(floatx4 a, floatx4 b, floatx4 c) {
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[0], b[0], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[1], b[1], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[2], b[2], c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[3], b[3], c, 0, 0, 0);
  return c;
}

// acc[i][j] += a[i] . b[j] over one 16-byte chunk per lane.  In fp32 the chunk takes four matrix
// instructions; they go round the accumulators, so that no two in a row depend on each other.
template <typename T, int NI, int NJ>
__device__ __forceinline__ void mma_block(const typename Vec16<T>::type (&a)[NI], const typename Vec16<T>::type (&b)[NJ],
                                          floatx4 (&acc)[NI][NJ]) {
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = mma16<T>(a[i], b[j], acc[i][j]);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
  }
}

// Thread index as a body sees it.  Inside the persistent kernel (COH != 0) the LDS-staged
// 64 x 64 contraction takes it through a statement the optimiser cannot see through: what it
// derives from it then stays inside the body instead of becoming an invariant of the
// work-item loop that is held in registers, or spilled at kernel entry (120 bytes per
// thread, 16 MB per launch), across every other operator's body.  Doing the same in every
// body costs 7 % (each tile recomputes its index arithmetic on the critical path); in this
// one it removes the spills and is 1-2 % faster on the CNN configs (measured).
template <int COH> __device__ __forceinline__ int body_thread() {
  int t = threadIdx.x;
  if constexpr (COH != 0) {
    asm volatile("" : "+v"(t));
    __builtin_assume(t >= 0 && t < 1024);
  }
  return t;
}

template <typename T, int BN, int BM, int WN, int WM, bool VEC, int COH, typename AR>
__device__ __forceinline__ void igemm_body(const AR &a, const Blk &b, unsigned char *lds) {
  typedef typename Vec16<T>::type V;
  typedef typename Vec16<T>::quad Q;
  constexpr int VE = Vec16<T>::N;
  constexpr int BKE = 4 * VE;              // K elements per slice
  constexpr int NT = WN * WM * 64;
  constexpr int ROWB = 80;                 // LDS row pitch in bytes (64 data + 16 pad)
  constexpr int CHW = BN * 4 / NT;         // 16-byte chunks of the weight tile per thread
  constexpr int CHX = BM * 4 / NT;
  constexpr int FN = BN / WN / 16, FM = BM / WM / 16;
  static_assert((BN * 4) % NT == 0 && (BM * 4) % NT == 0, "tile/threads mismatch");
  unsigned char (*smem)[(BN + BM) * ROWB] = (unsigned char (*)[(BN + BM) * ROWB])lds;   // [2][...]

  const int t = body_thread<COH>(), lane = t & 63, wave = t >> 6;
  const int wn0 = (wave % WN) * (BN / WN), wm0 = (wave / WN) * (BM / WM);
  const int m0 = b.x * BM, n0 = b.y * BN;
  constexpr bool CS = COH != 0;
  const T *__restrict__ x = (const T *)a.x;
  const T *__restrict__ w = (const T *)a.w;
  T *__restrict__ y = (T *)a.y;
  if (b.z) { x += (int64_t)b.z * a.a_bs; w += (int64_t)b.z * a.b_bs; y += (int64_t)b.z * a.y_bs; }
  const int kc = t & 3;                    // which 16-byte chunk of a 64-byte K slice
  const int row0 = t >> 2;                 // first tile row this thread moves
  constexpr int RSTEP = NT / 4;

  int ih0[CHX], iw0[CHX];
  const T *ximg[CHX];
  if (a.gather) {
#pragma unroll
    for (int i = 0; i < CHX; ++i) {
      const int m = m0 + row0 + i * RSTEP;
      const int img = m / a.HoWo, pix = m - img * a.HoWo;
      const int oh = pix / a.Wo, ow = pix - oh * a.Wo;
      ih0[i] = oh * a.sh - a.ph;
      iw0[i] = ow * a.sw - a.pw;
      ximg[i] = x + (int64_t)img * a.img_stride;
    }
  }
  // running decomposition of this thread's K position (vector path, gather only)
  int g_ci = 0, g_s = 0, g_r = 0;
  if (VEC && a.gather) {
    const int k = kc * VE;
    g_ci = k % a.Cin;
    const int rs = k / a.Cin;
    g_s = rs % a.kw;
    g_r = rs / a.kw;
  }

  V wreg[CHW], xreg[CHX];
  const V vzero = {};

  auto load_global = [&](int kt) {
    const int kbase = kt * BKE + kc * VE;
    // ---- pixel (im2col / matrix row) chunks
#pragma unroll
    for (int i = 0; i < CHX; ++i) {
      const int m = m0 + row0 + i * RSTEP;
      V v = vzero;
      if (VEC) {
        if (m < a.M && kbase < a.K) {
          if (!a.gather) {
            v = ldg<V>(x + (int64_t)m * a.lda + kbase);
          } else {
            const int ih = ih0[i] + g_r, iw = iw0[i] + g_s;
            if ((unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W)
              v = ldg<V>(ximg[i] + ((int64_t)ih * a.W + iw) * a.Cin + g_ci);
          }
        }
      } else {
        if (m < a.M) {
#pragma unroll
          for (int e = 0; e < VE; ++e) {
            const int k = kbase + e;
            if (k < a.K) {
              if (!a.gather) {
                v[e] = ldg<T>(x + (int64_t)m * a.lda + k);
              } else {
                const int ci = k % a.Cin, rs = k / a.Cin;
                const int ih = ih0[i] + rs / a.kw, iw = iw0[i] + rs % a.kw;
                if ((unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W)
                  v[e] = ldg<T>(ximg[i] + ((int64_t)ih * a.W + iw) * a.Cin + ci);
              }
            }
          }
        }
      }
      xreg[i] = v;
    }
    // ---- weight chunks
#pragma unroll
    for (int i = 0; i < CHW; ++i) {
      V v = vzero;
      if (!a.b_kmajor) {
        const int n = n0 + row0 + i * RSTEP;
        if (VEC) {
          if (n < a.N && kbase < a.K) v = ldg<V>(w + (int64_t)n * a.ldb + kbase);
        } else if (n < a.N) {
#pragma unroll
          for (int e = 0; e < VE; ++e)
            if (kbase + e < a.K) v[e] = ldg<T>(w + (int64_t)n * a.ldb + kbase + e);
        }
      } else {
        // operand stored [K][N]: a chunk runs along N at one K position
        const int c = t + i * NT;
        const int krow = c / (BN / VE), nch = c % (BN / VE);
        const int k = kt * BKE + krow, n = n0 + nch * VE;
        if (k < a.K) {
          if (VEC) {
            if (n < a.N) v = ldg<V>(w + (int64_t)k * a.ldb + n);
          } else {
#pragma unroll
            for (int e = 0; e < VE; ++e)
              if (n + e < a.N) v[e] = ldg<T>(w + (int64_t)k * a.ldb + n + e);
          }
        }
      }
      wreg[i] = v;
    }
    if (VEC && a.gather) {  // advance the running K decomposition by one slice
      g_ci += BKE;
      while (g_ci >= a.Cin) {
        g_ci -= a.Cin;
        if (++g_s == a.kw) { g_s = 0; ++g_r; }
      }
    }
  };

  auto store_lds = [&](int buf) {
    unsigned char *Wb = smem[buf];
    unsigned char *Xb = Wb + BN * ROWB;
#pragma unroll
    for (int i = 0; i < CHX; ++i) *(V *)(Xb + (row0 + i * RSTEP) * ROWB + kc * 16) = xreg[i];
#pragma unroll
    for (int i = 0; i < CHW; ++i) {
      if (!a.b_kmajor) {
        *(V *)(Wb + (row0 + i * RSTEP) * ROWB + kc * 16) = wreg[i];
      } else {
        const int c = t + i * NT;
        const int krow = c / (BN / VE), nch = c % (BN / VE);
#pragma unroll
        for (int e = 0; e < VE; ++e) *(T *)(Wb + (nch * VE + e) * ROWB + krow * (int)sizeof(T)) = wreg[i][e];
      }
    }
  };

  floatx4 acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  const int nk = (a.K + BKE - 1) / BKE;
  load_global(0);
  store_lds(0);
  __syncthreads();
  int buf = 0;
  for (int kt = 0; kt < nk; ++kt) {
    const bool more = kt + 1 < nk;
    if (more) load_global(kt + 1);
    {
      const unsigned char *Wb = smem[buf];
      const unsigned char *Xb = Wb + BN * ROWB;
      V af[FN], bf[FM];
#pragma unroll
      for (int i = 0; i < FN; ++i) af[i] = *(const V *)(Wb + (wn0 + i * 16 + (lane & 15)) * ROWB + (lane >> 4) * 16);
#pragma unroll
      for (int j = 0; j < FM; ++j) bf[j] = *(const V *)(Xb + (wm0 + j * 16 + (lane & 15)) * ROWB + (lane >> 4) * 16);
#pragma unroll
      for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = mma16<T>(af[i], bf[j], acc[i][j]);
    }
    if (more) store_lds(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }

  // ---- epilogue: alpha, bias, residual inputs, ReLU, convert, store
#pragma unroll
  for (int i = 0; i < FN; ++i) {
    const int n = n0 + wn0 + i * 16 + (lane >> 4) * 4;
#pragma unroll
    for (int j = 0; j < FM; ++j) {
      const int m = m0 + wm0 + j * 16 + (lane & 15);
      if (m >= a.M || n >= a.N) continue;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float r = acc[i][j][e] * a.alpha;
        if (n + e < a.N) {
          if (a.bias) r += a.bias[n + e];
          for (int q = 0; q < a.n_extra; ++q) r += (float)ldg<T>((const T *)a.extra[q] + (int64_t)m * a.N + n + e);
        }
        if (a.relu) r = fmaxf(r, 0.f);
        v[e] = r;
      }
      T *dst = y + (int64_t)m * a.ldy + n;
      if (n + 3 < a.N && ((uintptr_t)dst & (4 * sizeof(T) - 1)) == 0) {
        Q q4 = {(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
        stg<CS, Q>(dst, q4);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < a.N) stg<CS, T>(dst + e, (T)v[e]);
      }
    }
  }
}

// Workgroups are handed to the eight XCDs round-robin in launch order; each XCD has its
// own L2.  Remap the linear workgroup index so that every XCD works on a contiguous
// range of tiles (row tiles of one column tile first): neighbours that share operand
// rows then share an L2 instead of fetching them eight times.  No division: a wavefront issues
// an instruction every four to eight clocks, and forty of them ahead of the first load are a
// tenth of a microsecond of every launch.
__device__ __forceinline__ void xcd_tile(const Blk &b, uint32_t div_gx, int &tx, int &ty) {
  constexpr uint32_t kXcds = 8;
  if (!b.remap) { tx = b.x; ty = b.y; return; }
  const uint32_t nx = (uint32_t)b.gx, total = nx * (uint32_t)b.gy, lin = (uint32_t)b.lin;
  const uint32_t xcd = lin % kXcds, r = total % kXcds;
  const uint32_t tile = xcd * (total / kXcds) + (xcd < r ? xcd : r) + lin / kXcds;
  const uint32_t row = fast_div(tile, nx, div_gx);
  tx = (int)(tile - row * nx);
  ty = (int)row;
}

struct KPos { int ci, s, r; };

__device__ __forceinline__ void kpos_advance(KPos &p, int delta, int Cin, int kw) {
  p.ci += delta;
  while (p.ci >= Cin) {
    p.ci -= Cin;
    if (++p.s == kw) { p.s = 0; ++p.r; }
  }
}

// ---------------------------------------------------------------------------------
// Latency-oriented implicit GEMM for small problems (batch-1 convolutions, skinny
// GEMMs): a workgroup owns a 32 x 32 output tile and its WAVES wavefronts split K
// between them.  Every lane fetches its MFMA fragments straight from global memory
// (32 contiguous bytes per row and lane group, so four lane groups consume a whole
// 128-byte line), two 64-byte-deep K steps in flight at a time, no LDS and no
// barrier inside the K loop.  Partial tiles meet in LDS once, at the end, where 256
// threads apply the epilogue and write 8/16-byte pieces of output rows.
// ---------------------------------------------------------------------------------
template <typename T, int WAVES, int U, int COH, int NI, int NJ, typename AR>
__device__ __forceinline__ void igemm_direct_body(const AR &a, const Blk &b, unsigned char *lds) {
  typedef typename Vec16<T>::type V;
  typedef typename Vec16<T>::quad Q;
  constexpr int VE = Vec16<T>::N;
  constexpr int DS = 8 * VE;               // K elements per step: 4 lane groups x 2 chunks
  constexpr int PITCH = 36;                // floats per pixel row of a partial tile in LDS
  float (*part)[32][PITCH] = (float (*)[32][PITCH])lds;                                // [WAVES][32][PITCH]

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int grp = lane >> 4, r16 = lane & 15;
  int tile_x, tile_y;
  xcd_tile(b, a.div_gx, tile_x, tile_y);
  const int m0 = tile_x * (16 * NJ), n0 = tile_y * (16 * NI);
  constexpr bool CS = COH != 0;
  const T *__restrict__ x = (const T *)a.x;
  const T *__restrict__ w = (const T *)a.w;
  T *__restrict__ y = (T *)a.y;
  if (b.z) { x += (int64_t)b.z * a.a_bs; w += (int64_t)b.z * a.b_bs; y += (int64_t)b.z * a.y_bs; }

  const int nds = (a.K + DS - 1) / DS;
  const int per_wave = (nds + WAVES - 1) / WAVES;
  const int ds_begin = wave * per_wave;
  const int ds_end = min(nds, ds_begin + per_wave);

  // Rows are clamped into range and every load is unconditional (a load behind a branch
  // is waited for inside the branch).  Results of clamped rows are never stored; K
  // tails are cancelled by zeroing the weight fragment, padding taps by zeroing the
  // pixel fragment.
  const T *wrow[NI], *xrow[NJ], *ximg[NJ];
  int ih0[NJ], iw0[NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int n = min(n0 + i * 16 + r16, a.N - 1);
    wrow[i] = w + (int64_t)n * a.ldb;
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int m = min(m0 + j * 16 + r16, a.M - 1);
    xrow[j] = x + (int64_t)m * a.lda;
    const int img = m / a.HoWo, pix = m - img * a.HoWo;   // only meaningful when gathering
    const int oh = pix / a.Wo, ow = pix - oh * a.Wo;
    ih0[j] = oh * a.sh - a.ph;
    iw0[j] = ow * a.sw - a.pw;
    ximg[j] = x + (int64_t)img * a.img_stride;
  }
  KPos pos = {0, 0, 0};
  if (a.gather && ds_begin < ds_end) {
    const int k = ds_begin * DS + grp * 2 * VE;
    pos.ci = k % a.Cin;
    const int rs = k / a.Cin;
    pos.s = rs % a.kw;
    pos.r = rs / a.kw;
  }

  floatx4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const V vzero = {};

  // Epilogue operands of this thread's output piece (bias, residual inputs) are requested
  // before the K walk, so that their latency is hidden behind it.
  constexpr int PG = 4 * NI;               // four-channel pieces per tile row
  const int pm = t / PG, pn = (t % PG) * 4;
  const int m = m0 + pm, n = n0 + pn;
  const bool full = n + 3 < a.N;           // whole group of four channels inside the tensor
  const bool live = t < 16 * NJ * PG && m < a.M && n < a.N;
  floatx4 badd = {0.f, 0.f, 0.f, 0.f};
  if (live && a.bias) {
    if (full && ((uintptr_t)(a.bias + n) & 15) == 0) badd = *(const floatx4 *)(a.bias + n);
    else
      for (int e = 0; e < 4; ++e) if (n + e < a.N) badd[e] = a.bias[n + e];
  }
  if (live)
    for (int q = 0; q < a.n_extra; ++q) {
      const T *ex = (const T *)a.extra[q] + (int64_t)m * a.N + n;
      if (full && ((uintptr_t)ex & (4 * sizeof(T) - 1)) == 0) {
        const Q v = ldg<Q>(ex);
#pragma unroll
        for (int e = 0; e < 4; ++e) badd[e] += (float)v[e];
      } else {
        for (int e = 0; e < 4; ++e) if (n + e < a.N) badd[e] += (float)ldg<T>(ex + e);
      }
    }

  // One round = UU K steps requested together, then multiplied.  Full rounds of U steps,
  // then a shorter last round: steps past the end of a wavefront's K range would only
  // move bytes that are never used, and at these sizes the bytes set the time.
  auto round = [&](auto uu_tag, int ds) {
    constexpr int UU = decltype(uu_tag)::value;
    V wa[UU][NI][2], xb[UU][NJ][2];
    bool kok[UU][2], inb[UU][NJ][2];
#pragma unroll
    for (int u = 0; u < UU; ++u) {
      KPos pc = pos;                       // position of chunk 0 of this step
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int k = (ds + u) * DS + grp * 2 * VE + c * VE;
        kok[u][c] = k < a.K;
        const int ks = kok[u][c] ? k : 0;
#pragma unroll
        for (int i = 0; i < NI; ++i) wa[u][i][c] = ldg<V>(wrow[i] + ks);
        if (!a.gather) {
#pragma unroll
          for (int j = 0; j < NJ; ++j) xb[u][j][c] = ldg<V>(xrow[j] + ks);
        } else {
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            const int ih = ih0[j] + pc.r, iw = iw0[j] + pc.s;
            inb[u][j][c] = kok[u][c] && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            const int64_t off = inb[u][j][c] ? ((int64_t)ih * a.W + iw) * a.Cin + pc.ci : 0;
            xb[u][j][c] = ldg<V>(ximg[j] + off);
          }
          if (c == 0) kpos_advance(pc, VE, a.Cin, a.kw);
        }
      }
      if (a.gather) kpos_advance(pos, DS, a.Cin, a.kw);
    }
#pragma unroll
    for (int u = 0; u < UU; ++u)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int i = 0; i < NI; ++i) wa[u][i][c] = kok[u][c] ? wa[u][i][c] : vzero;
        if (a.gather) {
#pragma unroll
          for (int j = 0; j < NJ; ++j) xb[u][j][c] = inb[u][j][c] ? xb[u][j][c] : vzero;
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) acc[i][j] = mma16<T>(wa[u][i][c], xb[u][j][c], acc[i][j]);
      }
  };
  {
    int ds = ds_begin;
    for (; ds + U <= ds_end; ds += U) round(std::integral_constant<int, U>{}, ds);
    if constexpr (U > 2) {
      if (ds + 2 <= ds_end) { round(std::integral_constant<int, 2>{}, ds); ds += 2; }
    }
    if constexpr (U > 1) {
      if (ds < ds_end) round(std::integral_constant<int, 1>{}, ds);
    }
  }

  // ---- meet in LDS: lane holds channels n = i*16 + grp*4 + e of pixel m = j*16 + r16
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) *(floatx4 *)&part[wave][j * 16 + r16][i * 16 + grp * 4] = acc[i][j];
  __syncthreads();
  if (t < 16 * NJ * PG) {
    floatx4 sum = *(const floatx4 *)&part[0][pm][pn];
#pragma unroll
    for (int q = 1; q < WAVES; ++q) sum += *(const floatx4 *)&part[q][pm][pn];
    if (live) {
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float r = sum[e] * a.alpha + badd[e];
        v[e] = a.relu ? fmaxf(r, 0.f) : r;
      }
      T *dst = y + (int64_t)m * a.ldy + n;
      if (full && ((uintptr_t)dst & (4 * sizeof(T) - 1)) == 0) {
        Q q4 = {(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
        stg<CS, Q>(dst, q4);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < a.N) stg<CS, T>(dst + e, (T)v[e]);
      }
    }
  }
}

// ---------------------------------------------------------------------------------
// Operand staging of the two LDS-fed contractions below.
//
// Both walk K in steps of 128 bytes per row and move operand rows from global memory
// straight into workgroup memory (buffer_load_dwordx4 ... lds: no vector registers, no second
// instruction for the LDS write, many loads in flight per wavefront).  One instruction of a
// wavefront fills 1 KB: lane l writes 16 bytes at base + 16 * l, so it covers eight rows and
// lane l holds slot l % 8 of row l / 8.  The destination is fixed by the hardware, the source
// is free: a lane fetches the 16-byte chunk (slot ^ f(row)), which keeps eight adjacent lanes
// on one 128-byte line of memory and spreads the fragment reads of the matrix instructions
// (sixteen rows, one chunk each) over all banks.
//
// The buffer form checks every lane's offset against the operand's size and delivers zeros
// past it: padding taps, chunks past the end of K and rows past the end of the operand are
// given an offset no operand reaches (the host keeps operands below it) and cost no traffic.
// Offsets are 32-bit; the K position of a GEMM-shaped operand is the scalar offset, so a
// step takes no vector arithmetic at all, and a gathered row takes seven instructions.
// ---------------------------------------------------------------------------------
typedef int i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ i32x4 buffer_of(const void *base, uint32_t bytes) {
  const uint64_t p = (uint64_t)(uintptr_t)base;
  return i32x4{__builtin_amdgcn_readfirstlane((int)(uint32_t)p), __builtin_amdgcn_readfirstlane((int)((p >> 32) & 0xffffu)),
               __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};    // raw buffer, 32-bit data format
}
// Volatile statements keep their order among each other; what reads or writes the destination
// is kept apart from the load by the waits below, which clobber memory.  The compiler puts the
// wavefront's LDS address into m0 like any operand; one wait state between that and the load.
// (The builtin for this load schedules worse: GoogLeNet-like 119.4 against 121.8 us,
// Inception-v3-like 249.5 against 253.2, with m0 written here and not by the compiler.)
__device__ __forceinline__ void lds_load16(i32x4 buf, uint32_t offset, uint32_t soffset, uint32_t lds_base) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               : : "v"(offset), "s"(buf), "s"(soffset), "{m0}"(lds_base));
}
template <int N> __device__ __forceinline__ void wait_loads() {        // all but the N youngest vector loads
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}
template <int N> __device__ __forceinline__ void wait_loads_and_meet() {   // ... then the workgroup's barrier
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(N) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const unsigned char *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char *)p;
}
// Bytes of one wavefront's ring in igemm_split_body: S steps, or its partial tile.
constexpr int split_ring_bytes(int ni, int nj, int s) {
  const int ring = s * (ni + nj) * 16 * 128, part = nj * 16 * (ni * 16 + 4) * 4;
  return ring > part ? ring : part;
}
constexpr int log2_of(int v) { return v <= 1 ? 0 : 1 + log2_of(v / 2); }

// LW / LX: rows of the two operands this lane fetches per K step (one load instruction each).
// Steps must be requested in increasing order from kt0 on.
// FAR: the operands span more than 32-bit offsets reach; offsets then count from the tile's first row
// (gather: its first image).
template <typename T, int LW, int LX, bool FAR = false> struct Stager {
  static constexpr int VE = Vec16<T>::N, BKE = 8 * VE, ES = (int)sizeof(T);
  i32x4 wbuf, xbuf;
  uint32_t wo[LW], xo[LX];                // byte offset of this lane's chunk in K step 0 (gather: of tap 0, 0)
  int ih0[LX], iw0[LX];                   // gather: input position of tap 0, 0
  int kw0, kx0;                           // element offset of this lane's chunk inside a K step
  int ci, s, r;                           // gather: channel and tap of this lane's chunk in the next step
  int dci, ds, dr;                        // ... and how a step moves them
  int K, gather, H, W, Cin, kh, kw;       // the operator's, read once

  // Row i of an operand is group first + i * step of eight rows, row lane / 8 inside it.
  template <typename AR>
  __device__ __forceinline__ void init(const AR &a, const T *w, const T *x, int n0, int m0, int kt0, int first, int step,
                                       int lane, int wslot, int xslot) {
    const int l8 = lane >> 3;
    K = a.K; gather = a.gather; H = a.H; W = a.W; Cin = a.Cin; kh = a.kh; kw = a.kw;
    kw0 = wslot * VE;
    kx0 = xslot * VE;
    uint32_t wbytes = a.w_bytes, xbytes = a.x_bytes, wat = 0, xat = 0;   // wat, xat: what the offsets leave out, modulo 2^32
    if constexpr (FAR) {
      const int64_t wb = (int64_t)n0 * a.ldb, xb = gather ? (int64_t)(m0 / a.HoWo) * a.img_stride : (int64_t)m0 * a.lda;
      const int64_t we = (int64_t)(a.N - 1) * a.ldb + a.K;
      const int64_t xe = gather ? (int64_t)(a.M / a.HoWo) * a.img_stride : (int64_t)(a.M - 1) * a.lda + a.K;
      w += wb;
      x += xb;
      wat = (uint32_t)(wb * ES);
      xat = (uint32_t)(xb * ES);
      wbytes = (uint32_t)min((we - wb) * ES, (int64_t)kOperandMaxBytes);
      xbytes = (uint32_t)min((xe - xb) * ES, (int64_t)kOperandMaxBytes);
    }
    wbuf = buffer_of(w, wbytes);
    xbuf = buffer_of(x, xbytes);
#pragma unroll
    for (int i = 0; i < LW; ++i) {
      const int n = n0 + (first + i * step) * 8 + l8;
      wo[i] = n < a.N ? ((uint32_t)n * (uint32_t)a.ldb + (uint32_t)kw0) * ES - wat : kOperandMaxBytes;
    }
    if (!a.gather) {
#pragma unroll
      for (int i = 0; i < LX; ++i) {
        const int m = m0 + (first + i * step) * 8 + l8;
        xo[i] = m < a.M ? ((uint32_t)m * (uint32_t)a.lda + (uint32_t)kx0) * ES - xat : kOperandMaxBytes;
      }
    } else {
#pragma unroll
      for (int i = 0; i < LX; ++i) {
        const int m = m0 + (first + i * step) * 8 + l8;
        const int img = (int)fast_div(m, a.HoWo, a.div_HoWo), pix = m - img * a.HoWo;
        const int oh = (int)fast_div(pix, a.Wo, a.div_Wo), ow = pix - oh * a.Wo;
        ih0[i] = m < a.M ? oh * a.sh - a.ph : -(1 << 28);          // no tap of a row past the end is inside
        iw0[i] = ow * a.sw - a.pw;
        xo[i] = ((uint32_t)img * (uint32_t)a.img_stride + (uint32_t)(((oh * a.sh - a.ph) * a.W + iw0[i]) * a.Cin)) * ES - xat;
      }
      const int k = kt0 * BKE + kx0;
      const int rs = (int)fast_div(k, a.Cin, a.div_Cin);
      ci = k - rs * a.Cin;
      r = (int)fast_div(rs, a.kw, a.div_kw);
      s = rs - r * a.kw;
      const int drs = (int)fast_div(BKE, a.Cin, a.div_Cin);
      dci = BKE - drs * a.Cin;
      dr = (int)fast_div(drs, a.kw, a.div_kw);
      ds = drs - dr * a.kw;
    }
  }
  // Requests K step kt: operand rows to wl + i * pitch and xl + i * pitch.
  __device__ __forceinline__ void issue(int kt, uint32_t wl, uint32_t xl, uint32_t pitch) {
    const uint32_t kb = (uint32_t)kt * 128u;
    const bool wok = kt * BKE + kw0 < K;
#pragma unroll
    for (int i = 0; i < LW; ++i) lds_load16(wbuf, wok ? wo[i] : kOperandMaxBytes, kb, wl + i * pitch);
    if (gather) {
      const uint32_t tap = (__umul24(__umul24(r, W) + s, Cin) + ci) * ES;
      const bool ok = r < kh;
#pragma unroll
      for (int i = 0; i < LX; ++i) {
        const bool in = ok && (unsigned)(ih0[i] + r) < (unsigned)H && (unsigned)(iw0[i] + s) < (unsigned)W;
        lds_load16(xbuf, in ? xo[i] + tap : kOperandMaxBytes, 0, xl + i * pitch);
      }
      ci += dci; s += ds; r += dr;
      const bool wrap = ci >= Cin;
      ci -= wrap ? Cin : 0;
      s += wrap ? 1 : 0;
      const bool row = s >= kw;
      s -= row ? kw : 0;
      r += row ? 1 : 0;
    } else {
      const bool xok = kt * BKE + kx0 < K;
#pragma unroll
      for (int i = 0; i < LX; ++i) lds_load16(xbuf, xok ? xo[i] : kOperandMaxBytes, kb, xl + i * pitch);
    }
  }
};

// Epilogue of one run of four output channels: scale, bias, residual inputs, ReLU.  Global
// memory takes vectors at element alignment.
template <typename T> struct Run4;
template <> struct Run4<half_t> { typedef _Float16 type __attribute__((ext_vector_type(4), aligned(2))); };
template <> struct Run4<float> { typedef float type __attribute__((ext_vector_type(4), aligned(4))); };

template <typename T, typename AR>
__device__ __forceinline__ floatx4 finish4(const AR &a, floatx4 v, floatx4 bias, int m, int n) {
  typedef typename Run4<T>::type R;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = v[e] * a.alpha + bias[e];
  for (int q = 0; q < a.n_extra; ++q) {
    const T *ex = (const T *)a.extra[q] + (int64_t)m * a.N + n;
    if (n + 3 < a.N) {
      const R r = *(const R *)ex;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += (float)r[e];
    } else {
#pragma unroll
      for (int e = 0; e < 3; ++e) if (n + e < a.N) v[e] += (float)ex[e];
    }
  }
  if (a.relu) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
  }
  return v;
}
// Four biases from channel n on; zeros past the last channel and for an operator without bias
// (no branch: a load behind one is waited for at the end of the branch).
struct BiasRow {
  __amdgpu_buffer_rsrc_t buf;
  template <typename AR> __device__ __forceinline__ BiasRow(const AR &a)
      : buf(__builtin_amdgcn_make_buffer_rsrc((void *)a.bias, 0, a.bias ? a.N * 4 : 0, 0x00020000)) {}
  __device__ __forceinline__ floatx4 at(int n) const {
    return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(buf, n * 4, 0, 0));
  }
};
template <typename T, bool CS, typename AR>
__device__ __forceinline__ void store4(const AR &a, T *dst, floatx4 v, int n) {
  typedef typename Vec16<T>::quad Q;
  typedef typename Run4<T>::type R;
  const bool full = n + 3 < a.N && (!CS || ((uintptr_t)dst & (4 * sizeof(T) - 1)) == 0);   // atomic stores (8 bytes) need alignment
  if (full) {
    if constexpr (CS) stg<CS, Q>(dst, Q{(T)v[0], (T)v[1], (T)v[2], (T)v[3]});
    else *(R *)dst = R{(T)v[0], (T)v[1], (T)v[2], (T)v[3]};
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < a.N) stg<CS, T>(dst + e, (T)v[e]);
  }
}

// erf by the rational-times-exponential formula of Abramowitz & Stegun 7.1.26 (absolute error
// below 1.5e-7): one reciprocal, one exponential and five multiply-adds, against several
// dozen instructions of the correctly rounded library routine, which made GELU ALU-bound
// (128 MB: 60 us against 38 us for ReLU).  Used where the result is stored as fp16, whose
// spacing (2^-11 relative) is three orders of magnitude coarser than that error.
__device__ __forceinline__ float erf_as(float x) {
  const float ax = fabsf(x);
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * ax);
  const float poly = t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  const float r = 1.0f - poly * __expf(-ax * ax);
  return x < 0.f ? -r : r;
}

template <typename T> __device__ __forceinline__ float elt_apply(int op, float x) {
  if (op == 1) return fmaxf(x, 0.f);
  if (op == 2) {
    const float z = x * 0.70710678118654752f;
    return 0.5f * x * (1.0f + (std::is_same<T, half_t>::value ? erf_as(z) : erff(z)));
  }
  return x;
}

// Tail of a contraction: an element-wise operator that reads its result (TailArgs), computed on
// the values as they are stored: a launch (2.3 us) and a pass over the result less.  An input
// other than the result is requested before the K walk, like the bias, or before the first
// store.  Measured, fp16 (us, two launches -> one): 128 x 768 x 768 + sum 5.8 -> 3.7,
// 128 x 768 x 3072 + GELU 7.2 -> 5.4, 512 x 3072 x 768 + sum 11.3 -> 10.6.
struct NoTail {};
template <typename T, typename TL> struct Tail {
  typedef typename Vec16<T>::quad Q;
  static constexpr bool kOn = std::is_same<TL, TailArgs>::value;
  __amdgpu_buffer_rsrc_t first;            // the first input that is not the result; empty without one (see BiasRow)
  template <typename AR> __device__ __forceinline__ Tail(const AR &a, const TL &t) {
    if constexpr (kOn)
      first = __builtin_amdgcn_make_buffer_rsrc((void *)t.in[0], 0, t.n_in > 1 ? a.M * a.N * (int)sizeof(T) : 0, 0x00020000);
  }
  template <typename AR> __device__ __forceinline__ Q ahead(const AR &a, int m, int n) const {
    if constexpr (kOn) {
      const int at = (int)((uint32_t)(m * a.N + n) * (uint32_t)sizeof(T));
      if constexpr (sizeof(T) == 2) return __builtin_bit_cast(Q, __builtin_amdgcn_raw_buffer_load_b64(first, at, 0, 0));
      else return __builtin_bit_cast(Q, __builtin_amdgcn_raw_buffer_load_b128(first, at, 0, 0));
    }
    return Q{};
  }
  // v: four values of row m from column n on, before they are rounded; o: the first other input there.
  template <typename AR>
  static __device__ __forceinline__ void apply(const AR &a, const TL &t, floatx4 v, Q o, int m, int n) {
    if constexpr (kOn) {
      const int64_t at = (int64_t)m * a.N + n;
      floatx4 sum = {0.f, 0.f, 0.f, 0.f};
      for (int q = 0; q < t.n_in; ++q) {
        Q x;
        if (q == t.self) {
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = (T)v[e];
        } else {
          x = q - (q > t.self ? 1 : 0) == 0 ? o : *(const Q *)((const T *)t.in[1] + at);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) sum[e] += (float)x[e];
      }
      Q r;
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = (T)elt_apply<T>(t.op, sum[e]);
      *(Q *)((T *)t.y + at) = r;
    }
  }
};

// ---------------------------------------------------------------------------------
// Throughput-oriented contraction: BN columns x BM rows per workgroup of WN x WM
// wavefronts, a ring of S stages in workgroup memory, S - 1 stages requested ahead, one
// barrier per stage.
// What bounds it: per 128-byte stage of a 128 x 128 tile the matrix cores need 515 clocks,
// the fragment reads of four 64 x 64 wavefronts 512 clocks of LDS bandwidth and the loads
// 512 clocks at 64 bytes per clock; one workgroup alone does these in turn (1,500 clocks
// measured), two per compute unit overlap them.  Hence two stages (64 KB) and two workgroups
// per CU for the large tile, smaller tiles where there are too few large ones to give every
// CU two (see choose_tiles in plan.cpp).  Measured, fp16, eight 384 x 2496 x 3904 products in
// one launch: 960 TFLOP/s with 128 x 128 tiles, 731 with 64 x 128, 638 with 64 x 64; one
// 512 x 4096 x 4096 product 25.0 us (64 x 64, 687 TFLOP/s; the register-staged kernels that
// stood here: 42.8 us); convolution 3 x 3, 32 -> 64 channels, 16 images of 147 x 147: 152 -> 39 us.
// The rows of the weight operand are dealt to the fragments so that a lane's accumulators
// are 4 * FN consecutive channels of one row (wide stores, whole lines per wavefront).
// ---------------------------------------------------------------------------------
template <typename T, int BN, int BM, int WN, int WM, int S, int COH, bool FAR = false, typename AR, typename TL = NoTail>
__device__ __forceinline__ void igemm_tile_body(const AR &a, const Blk &b, unsigned char *lds, const TL &tail = TL{}) {
  typedef typename Vec16<T>::type V;
  constexpr int NW = WN * WM, STAGE = (BN + BM) * 128;
  constexpr int FN = BN / WN / 16, FM = BM / WM / 16;
  constexpr int LW = BN / 8 / NW, LX = BM / 8 / NW, L = LW + LX;
  constexpr int FB = 2 + log2_of(FN);      // row bit that tells apart rows whose low two bits repeat in a fragment
  static_assert(NW == 4 && BN % 32 == 0 && BM % 32 == 0 && (FN == 2 || FN == 4), "tile / wavefront mismatch");
  constexpr bool CS = COH != 0;

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int grp = lane >> 4, r16 = lane & 15;
  const int wn0 = (wave % WN) * (BN / WN), wm0 = (wave / WN) * (BM / WM);
  int tile_x, tile_y;
  xcd_tile(b, a.div_gx, tile_x, tile_y);
  const int m0 = tile_x * BM, n0 = tile_y * BN;
  const T *__restrict__ x = (const T *)a.x;
  const T *__restrict__ w = (const T *)a.w;
  T *__restrict__ y = (T *)a.y;
  if (b.z) { x += (int64_t)b.z * a.a_bs; w += (int64_t)b.z * a.b_bs; y += (int64_t)b.z * a.y_bs; }

  // Slot of chunk c of a row: c ^ fw(row) for the weights, c ^ (row & 7) for the other operand.
  auto fw = [](int row) { return (row & 3) | (((row >> FB) & 1) << 2); };
  Stager<T, LW, LX, FAR> st;
  st.init(a, w, x, n0, m0, 0, wave, NW, lane, (lane & 7) ^ fw(wave * 8 + (lane >> 3)), (lane & 7) ^ (lane >> 3));
  const uint32_t base = lds_address(lds) + wave * 1024;
  auto issue = [&](int kt, int slot) {
    st.issue(kt, base + slot * STAGE, base + slot * STAGE + BN * 128, NW * 1024);
  };

  floatx4 acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int nst = (a.K + Stager<T, LW, LX, FAR>::BKE - 1) / Stager<T, LW, LX, FAR>::BKE;
#pragma unroll
  for (int s = 0; s < S - 1; ++s)
    if (s < nst) issue(s, s);
  const int nrun = n0 + wn0 + grp * 4 * FN;            // this lane's first output channel
  const BiasRow bias(a);
  floatx4 bv[FN];
#pragma unroll
  for (int i = 0; i < FN; ++i) bv[i] = bias.at(nrun + i * 4);

  const int wrow = wn0 + (r16 >> 2) * (4 * FN) + (r16 & 3);
  int slot = 0, ahead = S - 1;
#pragma nounroll
  for (int kt = 0; kt < nst; ++kt) {
    // Stage kt has arrived once at most the S - 2 younger ones are in flight; behind the
    // barrier everybody's part of it has, and nobody reads the slot that is refilled next.
    if (kt + S - 2 < nst) wait_loads_and_meet<(S - 2) * L>();
    else wait_loads_and_meet<0>();
    if (kt + S - 1 < nst) issue(kt + S - 1, ahead);
    const unsigned char *Wb = lds + slot * STAGE, *Xb = Wb + BN * 128;
    V af[2][FN], bf[2][FM];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < FN; ++i) {
        const int row = wrow + i * 4;
        af[ks][i] = *(const V *)(Wb + row * 128 + (((ks * 4 + grp) ^ fw(row)) * 16));
      }
#pragma unroll
      for (int j = 0; j < FM; ++j) {
        const int row = wm0 + j * 16 + r16;
        bf[ks][j] = *(const V *)(Xb + row * 128 + (((ks * 4 + grp) ^ (row & 7)) * 16));
      }
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) mma_block<T>(af[ks], bf[ks], acc);
    slot = slot == S - 1 ? 0 : slot + 1;
    ahead = ahead == S - 1 ? 0 : ahead + 1;
  }

  typedef V VU __attribute__((aligned(sizeof(T))));
  typedef Tail<T, TL> After;
  typename After::Q ov[FN][FM];                        // what the tail adds, all requested before the first store
  if constexpr (After::kOn) {
    const After after(a, tail);
    if (tail.n_in > 1) {
#pragma unroll
      for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int i = 0; i < FN; ++i) ov[i][j] = after.ahead(a, m0 + wm0 + j * 16 + r16, nrun + i * 4);
    }
  }
#pragma unroll
  for (int j = 0; j < FM; ++j) {
    const int m = m0 + wm0 + j * 16 + r16;
    if (m >= a.M) continue;
    T *dst = y + (int64_t)m * a.ldy + nrun;
#pragma unroll
    for (int i = 0; i < FN; i += VecRun<T>::N) {
      const int n = nrun + i * 4;
      if (n >= a.N) break;
      if constexpr (VecRun<T>::N == 2) {               // eight halves: one 16-byte store
        const floatx4 lo = finish4<T>(a, acc[i][j], bv[i], m, n);
        const floatx4 hi = finish4<T>(a, acc[i + 1][j], bv[i + 1], m, n + 4);
        After::apply(a, tail, lo, ov[i][j], m, n);
        if (n + 4 < a.N) After::apply(a, tail, hi, ov[i + 1][j], m, n + 4);
        if (n + 7 < a.N) {
          V o;
#pragma unroll
          for (int e = 0; e < 4; ++e) { o[e] = (T)lo[e]; o[4 + e] = (T)hi[e]; }
          if constexpr (CS) stg<CS, V>(dst + i * 4, o);
          else *(VU *)(dst + i * 4) = o;
        } else {
          store4<T, CS>(a, dst + i * 4, lo, n);
          store4<T, CS>(a, dst + i * 4 + 4, hi, n + 4);
        }
      } else {
        const floatx4 v = finish4<T>(a, acc[i][j], bv[i], m, n);
        After::apply(a, tail, v, ov[i][j], m, n);
        store4<T, CS>(a, dst + i * 4, v, n);
      }
    }
  }
}

// ---------------------------------------------------------------------------------
// Latency-oriented contraction (batch-1 convolutions, skinny GEMMs): one 16 NI columns x
// 16 NJ rows tile per workgroup, K shared out between its four wavefronts in whole 128-byte
// steps.  Every wavefront stages its own steps in its own ring of S slots and waits for its
// own loads only: no barrier until the partial tiles meet, each in its wavefront's ring.
// What bounds it: with few tiles the load rate of one compute unit, which is why a small
// problem takes small tiles on many CUs; with many, the bytes (a 32 x 32 tile moves twice
// the operand bytes per multiply-add of a 64 x 64 one).  Measured, isolated fp16 products
// (us; register-staged kernels that stood here before -> now, with the tile taken):
// 128 x 768 x 3072 7.5 -> 5.3 (32 x 32), 512 x 768 x 3072 13.8 -> 7.9 (64 x 32),
// 256 x 2048 x 2048 13.5 -> 6.8 (64 x 32), 64 x 4096 x 4096 13.6 -> 8.2 (32 x 32),
// 256 x 4096 x 4096 30.3 -> 15.8 (64 x 64).
// ---------------------------------------------------------------------------------
template <typename T, int NI, int NJ, int S, int COH, typename AR, typename TL = NoTail>
__device__ __forceinline__ void igemm_split_body(const AR &a, const Blk &b, unsigned char *lds, const TL &tail = TL{}) {
  typedef typename Vec16<T>::type V;
  constexpr int WAVES = 4, BN = 16 * NI, BM = 16 * NJ, STEP = (BN + BM) * 128;
  constexpr int PITCH = BN + 4;            // floats per row of a partial tile
  constexpr int RING = split_ring_bytes(NI, NJ, S);
  constexpr int LW = BN / 8, LX = BM / 8, L = LW + LX;
  constexpr bool CS = COH != 0;

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int grp = lane >> 4, r16 = lane & 15;
  int tile_x, tile_y;
  xcd_tile(b, a.div_gx, tile_x, tile_y);
  const int m0 = tile_x * BM, n0 = tile_y * BN;
  const T *__restrict__ x = (const T *)a.x;
  const T *__restrict__ w = (const T *)a.w;
  T *__restrict__ y = (T *)a.y;
  if (b.z) { x += (int64_t)b.z * a.a_bs; w += (int64_t)b.z * a.b_bs; y += (int64_t)b.z * a.y_bs; }

  const int nst = (a.K + Stager<T, LW, LX>::BKE - 1) / Stager<T, LW, LX>::BKE;
  const int k_begin = nst * wave / WAVES, k_end = nst * (wave + 1) / WAVES;
  Stager<T, LW, LX> st;
  const int cslot = (lane & 7) ^ (lane >> 3);
  st.init(a, w, x, n0, m0, k_begin, 0, 1, lane, cslot, cslot);
  unsigned char *ring = lds + wave * RING;
  const uint32_t base = lds_address(ring);
  auto issue = [&](int kt, int slot) { st.issue(kt, base + slot * STEP, base + slot * STEP + BN * 128, 1024); };
#pragma unroll
  for (int s = 0; s < S; ++s)
    if (k_begin + s < k_end) issue(k_begin + s, s);

  floatx4 acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  // Bias of this thread's output pieces, requested before the K walk.
  constexpr int PG = 4 * NI, PIECES = (BM * PG + 255) / 256;   // four-channel pieces per row, per thread
  const BiasRow bias(a);
  const Tail<T, TL> after(a, tail);
  floatx4 bv[PIECES];
  typename Tail<T, TL>::Q tv[PIECES];
#pragma unroll
  for (int p = 0; p < PIECES; ++p) {
    const int idx = t + p * 256, n = n0 + (idx % PG) * 4;
    bv[p] = bias.at(n);
    tv[p] = after.ahead(a, m0 + idx / PG, n);
  }
  int slot = 0;
#pragma nounroll
  for (int kt = k_begin; kt < k_end; ++kt) {
    if (kt + S - 1 < k_end) wait_loads<(S - 1) * L>();
    else wait_loads<0>();
    const unsigned char *Wb = ring + slot * STEP, *Xb = Wb + BN * 128;
    V af[2][NI], bf[2][NJ];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int c = ((ks * 4 + grp) ^ (r16 & 7)) * 16;
#pragma unroll
      for (int i = 0; i < NI; ++i) af[ks][i] = *(const V *)(Wb + (i * 16 + r16) * 128 + c);
#pragma unroll
      for (int j = 0; j < NJ; ++j) bf[ks][j] = *(const V *)(Xb + (j * 16 + r16) * 128 + c);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");     // the slot has been read: it may be refilled
    if (kt + S < k_end) issue(kt + S, slot);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) mma_block<T>(af[ks], bf[ks], acc);
    slot = slot == S - 1 ? 0 : slot + 1;
  }

  // ---- partial tiles meet: lane holds channels n = i*16 + grp*4 + e of row m = j*16 + r16
  float *part = (float *)ring;
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) *(floatx4 *)(part + (j * 16 + r16) * PITCH + i * 16 + grp * 4) = acc[i][j];
  __syncthreads();
#pragma unroll
  for (int p = 0; p < PIECES; ++p) {
    const int idx = t + p * 256;
    const int pm = idx / PG, pn = (idx % PG) * 4;
    const int m = m0 + pm, n = n0 + pn;
    if (idx >= BM * PG || m >= a.M || n >= a.N) continue;
    const unsigned char *at = lds + (pm * PITCH + pn) * 4;
    floatx4 sum = *(const floatx4 *)at;
#pragma unroll
    for (int q = 1; q < WAVES; ++q) sum += *(const floatx4 *)(at + q * RING);
    const floatx4 v = finish4<T>(a, sum, bv[p], m, n);
    Tail<T, TL>::apply(a, tail, v, tv[p], m, n);
    store4<T, CS>(a, y + (int64_t)m * a.ldy + n, v, n);
  }
}

// Matrix-vector shaped GEMM (M <= kGemvMaxM rows): one wavefront per output column,
// 16-byte loads along K, shuffle reduction.  Weight-bandwidth bound by construction.
template <typename T, int COH, typename AR>
__device__ __forceinline__ void gemv_body(const AR &a, const Blk &b, unsigned char *lds) {
  typedef typename Vec16<T>::type V;
  constexpr int VE = Vec16<T>::N;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n = b.x * 4 + wave;
  if (n >= a.N) return;
  constexpr bool CS = COH != 0;
  const T *__restrict__ x = (const T *)a.x;
  const T *__restrict__ wr = (const T *)a.w + (int64_t)n * a.ldb;
  float acc[kGemvMaxM] = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = lane * VE; k0 < a.K; k0 += 64 * VE) {
    const V wv = ldg<V>(wr + k0);
#pragma unroll
    for (int m = 0; m < kGemvMaxM; ++m) {
      if (m < a.M) {
        const V xv = ldg<V>(x + (int64_t)m * a.lda + k0);
#pragma unroll
        for (int e = 0; e < VE; ++e) acc[m] += (float)wv[e] * (float)xv[e];
      }
    }
  }
#pragma unroll
  for (int m = 0; m < kGemvMaxM; ++m)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc[m] += __shfl_xor(acc[m], off, 64);
  if (lane == 0) {
    T *y = (T *)a.y;
    for (int m = 0; m < a.M; ++m) {
      float r = acc[m] * a.alpha;
      if (a.bias) r += a.bias[n];
      for (int q = 0; q < a.n_extra; ++q) r += (float)ldg<T>((const T *)a.extra[q] + (int64_t)m * a.N + n);
      if (a.relu) r = fmaxf(r, 0.f);
      stg<CS, T>(y + (int64_t)m * a.ldy + n, (T)r);
    }
  }
}

// ---------------------------------------------------------------------------------
// Pooling over [H][W][C]: one thread per output pixel and channel chunk.
// What bounds it: at batch 1 the latency of one pass (index arithmetic, one round of loads),
// at large batches vector instructions, not bytes: nine taps of eight halves.  Hence no
// division (the host hands over reciprocals), 32-bit offsets from a uniform base, positions
// clamped into the image instead of a select per tap and channel (the nearest valid position
// of a tap outside the image lies inside the window too, so a maximum does not see it twice;
// an average zeroes the whole chunk), packed half maxima, and conversion and addition of an
// average in one instruction.  Measured, fp16: 64 channels of 112 x 112
// to 56 x 56 3.65 -> 2.43 us (an empty launch: 2.2), 16 images of 256 x 35 x 35 averaged 13.0 ->
// 6.9 us, 16 of 64 x 147 x 147 to 73 x 73 14.5 -> 12.0 us (4.6 TB/s).
// ---------------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ T lane_max(T a, T b) { return __builtin_elementwise_max(a, b); }

template <typename T, int VE, bool AVG, typename AR>
__device__ __forceinline__ void pool_window(const AR &a, uint32_t xoff, int ih0, int iw0, T *o) {
  typedef T V __attribute__((ext_vector_type(VE)));
  const unsigned char *__restrict__ x = (const unsigned char *)a.x;
  const uint32_t pitch = (uint32_t)a.C * (uint32_t)sizeof(T);
  V best;
  float acc[VE], one = 1.0f;
  asm volatile("" : "+v"(one));                          // kept unknown: conversion and addition stay one fused multiply-add
#pragma unroll
  for (int e = 0; e < VE; ++e) { best[e] = (T)-INFINITY; acc[e] = 0.f; }
  auto at = [&](int ih, int iw, bool &ok) {
    const int ch = min(max(ih, 0), a.H - 1), cw = min(max(iw, 0), a.W - 1);
    ok = ch == ih && cw == iw;
    return xoff + (uint32_t)(ch * a.W + cw) * pitch;
  };
  auto fold = [&](V v, bool ok) {
    if constexpr (AVG) {
      const V zero = {};
      v = ok ? v : zero;
#pragma unroll
      for (int e = 0; e < VE; ++e) acc[e] = __builtin_fmaf((float)v[e], one, acc[e]);
    } else {
      best = lane_max(best, v);
    }
  };
  if (a.kh == 3 && a.kw == 3) {                          // all nine taps in flight before the first use
    V v[9];
    bool ok[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) v[q] = *(const V *)(x + at(ih0 + q / 3, iw0 + q % 3, ok[q]));
#pragma unroll
    for (int q = 0; q < 9; ++q) fold(v[q], ok[q]);
  } else {
    for (int i = 0; i < a.kh; ++i)
      for (int j = 0; j < a.kw; ++j) {
        bool ok;
        const V v = *(const V *)(x + at(ih0 + i, iw0 + j, ok));
        fold(v, ok);
      }
  }
  const float scale = 1.0f / (float)(a.kh * a.kw);
#pragma unroll
  for (int e = 0; e < VE; ++e) o[e] = AVG ? (T)(acc[e] * scale) : best[e];
}

template <typename T, int VE, int COH, typename AR>
__device__ __forceinline__ void pool_body(const AR &a, const Blk &b, unsigned char *lds) {
  typedef T V __attribute__((ext_vector_type(VE)));
  constexpr bool CS = COH != 0;
  const uint32_t cch = (uint32_t)(a.C / VE);
  int64_t pix64;
  int cc, img, oh, ow;
  if (a.items) {                                         // everything within reach of 32-bit offsets
    const uint32_t item = (uint32_t)b.x * 256u + threadIdx.x;
    if (item >= a.items) return;
    const uint32_t pix = fast_div(item, cch, a.div_cch);
    cc = (int)(item - pix * cch);
    img = (int)fast_div(pix, a.Ho * a.Wo, a.div_HoWo);
    const uint32_t ipix = pix - (uint32_t)(img * a.Ho * a.Wo);
    oh = (int)fast_div(ipix, a.Wo, a.div_Wo);
    ow = (int)ipix - oh * a.Wo;
    V o;
    const uint32_t xoff = ((uint32_t)img * (uint32_t)(a.H * a.W * a.C) + (uint32_t)cc * VE) * (uint32_t)sizeof(T);
    if (a.is_avg) pool_window<T, VE, true>(a, xoff, oh * a.sh - a.ph, ow * a.sw - a.pw, (T *)&o);
    else pool_window<T, VE, false>(a, xoff, oh * a.sh - a.ph, ow * a.sw - a.pw, (T *)&o);
    T *dst = (T *)((unsigned char *)a.y + (pix * (uint32_t)a.C + (uint32_t)cc * VE) * (uint32_t)sizeof(T));
    if constexpr (VE > 1) stg<CS, typename Vec16<T>::type>(dst, __builtin_bit_cast(typename Vec16<T>::type, o));
    else stg<CS, T>(dst, o[0]);
    return;
  }
  const int64_t item = (int64_t)b.x * 256 + threadIdx.x;
  if (item >= (int64_t)a.B * a.Ho * a.Wo * cch) return;
  cc = (int)(item % cch);
  pix64 = item / cch;                                    // output pixel over all images
  img = (int)(pix64 / ((int64_t)a.Ho * a.Wo));
  const int ipix = (int)(pix64 - (int64_t)img * a.Ho * a.Wo);
  ow = ipix % a.Wo; oh = ipix / a.Wo;
  const T *__restrict__ x = (const T *)a.x + (int64_t)img * a.H * a.W * a.C + cc * VE;
  float acc[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) acc[e] = a.is_avg ? 0.f : -INFINITY;
  for (int i = 0; i < a.kh; ++i)
    for (int j = 0; j < a.kw; ++j) {
      const int ih = oh * a.sh - a.ph + i, iw = ow * a.sw - a.pw + j;
      if ((unsigned)ih >= (unsigned)a.H || (unsigned)iw >= (unsigned)a.W) continue;
      const V v = *(const V *)(x + ((int64_t)ih * a.W + iw) * a.C);
#pragma unroll
      for (int e = 0; e < VE; ++e) acc[e] = a.is_avg ? acc[e] + (float)v[e] : fmaxf(acc[e], (float)v[e]);
    }
  const float scale = a.is_avg ? 1.0f / (float)(a.kh * a.kw) : 1.0f;
  T *dst = (T *)a.y + pix64 * a.C + cc * VE;
  V o;
#pragma unroll
  for (int e = 0; e < VE; ++e) o[e] = (T)(a.is_avg ? acc[e] * scale : acc[e]);
  if constexpr (VE > 1) stg<CS, typename Vec16<T>::type>(dst, __builtin_bit_cast(typename Vec16<T>::type, o));
  else stg<CS, T>(dst, o[0]);
}

// Global average pool over [HW][C].  Vector form: two threads hold a pixel's 16-byte chunks,
// the others take further pixels (128 of them at once); four pixels per thread in flight;
// slices meet by shuffles inside a wavefront and in LDS across the four.  A serial chain of loads
// bounds it, so an image of many pixels takes two chunks per pixel (160 channels of 28 x 28: 8.1
// -> 3.5 us).  Scalar form, for few pixels or odd channel counts: 64 channels x 4 pixel slices.
template <typename T, int COH, typename AR>
__device__ __forceinline__ void gap_body(const AR &a, const Blk &b, unsigned char *lds) {
  typedef typename Vec16<T>::type V;
  constexpr int VE = Vec16<T>::N;
  constexpr bool CS = COH != 0;
  const T *__restrict__ x = (const T *)a.x + (int64_t)b.y * a.HW * a.C;
  if (a.vec) {
    float (*part)[2 * VE] = (float (*)[2 * VE])lds;                                    // [4][chunks per pixel * VE]
    constexpr int lp = kGapShare;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int chunk = threadIdx.x & ((1 << lp) - 1), slices = 256 >> lp;
    const int c = ((b.x << lp) + chunk) * VE;
    float s[VE];
#pragma unroll
    for (int e = 0; e < VE; ++e) s[e] = 0.f;
    if (c < a.C) {
      const T *xc = x + c;
      for (int p = threadIdx.x >> lp; p < a.HW; p += 4 * slices) {
        V v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = ldg<V>(xc + (int64_t)min(p + q * slices, a.HW - 1) * a.C);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (p + q * slices < a.HW)
#pragma unroll
            for (int e = 0; e < VE; ++e) s[e] += (float)v[q][e];
      }
    }
    for (int off = 32; off >= 1 << lp; off >>= 1)
#pragma unroll
      for (int e = 0; e < VE; ++e) s[e] += __shfl_xor(s[e], off, 64);
    if (lane < 1 << lp)
#pragma unroll
      for (int e = 0; e < VE; ++e) part[wave][chunk * VE + e] = s[e];
    __syncthreads();
    if (threadIdx.x < 1 << lp && c < a.C) {
      V o;
#pragma unroll
      for (int e = 0; e < VE; ++e) {
        const int i = chunk * VE + e;
        o[e] = (T)((part[0][i] + part[1][i] + part[2][i] + part[3][i]) / (float)a.HW);
      }
      stg<CS, V>((T *)a.y + (int64_t)b.y * a.C + c, o);
    }
    return;
  }
  float (*part)[64] = (float (*)[64])lds;                                              // [4][64]
  const int cl = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int c = b.x * 64 + cl;
  float s = 0.f;
  if (c < a.C) {
    int p = slice;
    for (; p + 12 < a.HW; p += 16) {
      const float v0 = (float)ldg<T>(x + (int64_t)p * a.C + c), v1 = (float)ldg<T>(x + (int64_t)(p + 4) * a.C + c);
      const float v2 = (float)ldg<T>(x + (int64_t)(p + 8) * a.C + c), v3 = (float)ldg<T>(x + (int64_t)(p + 12) * a.C + c);
      s += (v0 + v1) + (v2 + v3);
    }
    for (; p < a.HW; p += 4) s += (float)ldg<T>(x + (int64_t)p * a.C + c);
  }
  part[slice][cl] = s;
  __syncthreads();
  if (slice == 0 && c < a.C)
    stg<CS, T>((T *)a.y + (int64_t)b.y * a.C + c, (T)((part[0][cl] + part[1][cl] + part[2][cl] + part[3][cl]) / (float)a.HW));
}

// ---------------------------------------------------------------------------------
// Row-wise LayerNorm / softmax of the summed inputs.  G lanes share a row (a
// wavefront, or the 256-thread workgroup); the row lives in registers between the
// statistics passes, so HBM sees one read per input and one write.
// ---------------------------------------------------------------------------------
template <int G, bool IS_MAX>
__device__ __forceinline__ float group_reduce(float v, float *scratch) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float o = __shfl_xor(v, off, 64);
    v = IS_MAX ? fmaxf(v, o) : v + o;
  }
  if (G > 64) {
    const int wave = threadIdx.x >> 6;
    __syncthreads();                    // scratch may still be read from a previous reduction
    if ((threadIdx.x & 63) == 0) scratch[wave] = v;
    __syncthreads();
    v = scratch[0];
#pragma unroll
    for (int i = 1; i < G / 64; ++i) v = IS_MAX ? fmaxf(v, scratch[i]) : v + scratch[i];
  }
  return v;
}

template <typename T, bool IS_LN, int G, int MAXCH, int COH, typename AR>
__device__ __forceinline__ void row_cached_body(const AR &a, const Blk &b, unsigned char *lds) {
  typedef typename Vec16<T>::type V;
  constexpr int VE = Vec16<T>::N;
  float *scratch = (float *)lds;                                                       // [4]
  constexpr bool CS = COH != 0;
  const int gl = threadIdx.x % G;
  const int row = b.x * (256 / G) + threadIdx.x / G;
  if (G == 64 && row >= a.rows) return;          // whole wavefront leaves together
  float v[MAXCH][VE];
  const int64_t base = (int64_t)row * a.cols;
#pragma unroll
  for (int c = 0; c < MAXCH; ++c) {
    const int col = (c * G + gl) * VE;
#pragma unroll
    for (int e = 0; e < VE; ++e) v[c][e] = 0.f;
    if (col < a.cols) {
      for (int q = 0; q < a.n_in; ++q) {
        const V t = ldg<V>((const T *)a.in[q] + base + col);
#pragma unroll
        for (int e = 0; e < VE; ++e) v[c][e] += (float)t[e];
      }
    }
  }
  if (IS_LN) {
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < MAXCH; ++c)
      if ((c * G + gl) * VE < a.cols)
#pragma unroll
        for (int e = 0; e < VE; ++e) s += v[c][e];
    const float mean = group_reduce<G, false>(s, scratch) / (float)a.cols;
    float q = 0.f;
#pragma unroll
    for (int c = 0; c < MAXCH; ++c)
      if ((c * G + gl) * VE < a.cols)
#pragma unroll
        for (int e = 0; e < VE; ++e) { const float d = v[c][e] - mean; q += d * d; }
    const float var = group_reduce<G, false>(q, scratch) / (float)a.cols;
    const float rstd = 1.0f / sqrtf(var + a.eps);
#pragma unroll
    for (int c = 0; c < MAXCH; ++c)
#pragma unroll
      for (int e = 0; e < VE; ++e) v[c][e] = (v[c][e] - mean) * rstd;
  } else {
    float mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < MAXCH; ++c)
      if ((c * G + gl) * VE < a.cols)
#pragma unroll
        for (int e = 0; e < VE; ++e) mx = fmaxf(mx, v[c][e]);
    mx = group_reduce<G, true>(mx, scratch);
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < MAXCH; ++c)
      if ((c * G + gl) * VE < a.cols)
#pragma unroll
        for (int e = 0; e < VE; ++e) { v[c][e] = expf(v[c][e] - mx); s += v[c][e]; }
    const float inv = 1.0f / group_reduce<G, false>(s, scratch);
#pragma unroll
    for (int c = 0; c < MAXCH; ++c)
#pragma unroll
      for (int e = 0; e < VE; ++e) v[c][e] *= inv;
  }
#pragma unroll
  for (int c = 0; c < MAXCH; ++c) {
    const int col = (c * G + gl) * VE;
    if (col < a.cols) {
      V o;
#pragma unroll
      for (int e = 0; e < VE; ++e) o[e] = (T)v[c][e];
      stg<CS, V>((T *)a.y + base + col, o);
    }
  }
}

// Any width / alignment: one workgroup per row, scalar accesses, inputs re-read per pass.
template <typename T, bool IS_LN, int COH, typename AR>
__device__ __forceinline__ void row_generic_body(const AR &a, const Blk &b, unsigned char *lds) {
  float *scratch = (float *)lds;                                                       // [4]
  constexpr bool CS = COH != 0;
  const int64_t base = (int64_t)b.x * a.cols;
  auto value = [&](int col) {
    float s = 0.f;
    for (int q = 0; q < a.n_in; ++q) s += (float)ldg<T>((const T *)a.in[q] + base + col);
    return s;
  };
  float p1 = IS_LN ? 0.f : -INFINITY;
  for (int col = threadIdx.x; col < a.cols; col += 256) p1 = IS_LN ? p1 + value(col) : fmaxf(p1, value(col));
  const float r1 = IS_LN ? group_reduce<256, false>(p1, scratch) / (float)a.cols : group_reduce<256, true>(p1, scratch);
  float p2 = 0.f;
  for (int col = threadIdx.x; col < a.cols; col += 256) {
    const float d = value(col) - r1;
    p2 += IS_LN ? d * d : expf(d);
  }
  const float r2 = group_reduce<256, false>(p2, scratch);
  const float k = IS_LN ? 1.0f / sqrtf(r2 / (float)a.cols + a.eps) : 1.0f / r2;
  for (int col = threadIdx.x; col < a.cols; col += 256) {
    const float d = value(col) - r1;
    stg<CS, T>((T *)a.y + base + col, (T)(IS_LN ? d * k : expf(d) * k));
  }
}

// ---------------------------------------------------------------------------------
// Element-wise f(sum of inputs) and channel/column concatenation.
// ---------------------------------------------------------------------------------
template <typename T, int VE, int COH, typename AR>
__device__ __forceinline__ void elt_body(const AR &a, const Blk &b, unsigned char *lds) {
  constexpr bool CS = COH != 0;
  const int64_t i = ((int64_t)b.x * 256 + threadIdx.x) * VE;
  if (i >= a.n) return;
  float s[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) s[e] = 0.f;
  for (int q = 0; q < a.n_in; ++q) {
    T v[VE];
    const T *src = (const T *)a.in[q] + i;
    if constexpr (VE > 1) *(typename Vec16<T>::type *)v = ldg<typename Vec16<T>::type>(src);
    else v[0] = ldg<T>(src);
#pragma unroll
    for (int e = 0; e < VE; ++e) s[e] += (float)v[e];
  }
  T o[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) o[e] = (T)elt_apply<T>(a.op, s[e]);
  T *dst = (T *)a.y + i;
  if constexpr (VE > 1) {
    typedef typename Vec16<T>::type V;
    stg<CS, V>(dst, *(const V *)o);
    if constexpr (!CS) {
      if (a.also) {
        const uint32_t item = (uint32_t)(i / VE), cch = (uint32_t)a.also_cols / VE, r = fast_div(item, cch, a.div_also);
        *(V *)((T *)a.also + (int64_t)r * a.also_pitch + (item - r * cch) * VE) = *(const V *)o;
      }
    }
  } else {
    stg<CS, T>(dst, o[0]);
  }
}

template <typename T, int VE, int COH, typename AR>
__device__ __forceinline__ void concat_body(const AR &a, const Blk &b, unsigned char *lds) {
  constexpr bool CS = COH != 0;
  const int q = b.y;
  const int cch = a.cols[q] / VE;
  const int64_t item = (int64_t)b.x * 256 + threadIdx.x;
  if (item >= (int64_t)a.rows * cch) return;
  const int64_t r = item >> 32 ? item / cch : (int64_t)fast_div((uint32_t)item, cch, a.div_cols[q]);   // no long division on the way
  const int c = (int)(item - r * cch) * VE;
  const T *src = (const T *)a.in[q] + r * a.cols[q] + c;
  T *dst = (T *)a.y + r * a.out_cols + a.col_off[q] + c;
  if constexpr (VE > 1) stg<CS, typename Vec16<T>::type>(dst, ldg<typename Vec16<T>::type>(src));
  else stg<CS, T>(dst, ldg<T>(src));
}

#include "attention.h"

}  // namespace opara

using namespace opara;

// Workgroup-shared memory each body needs (bytes).
constexpr int lds_igemm(int bn, int bm) { return 2 * (bn + bm) * 80; }
constexpr int lds_tile(int bn, int bm, int stages) { return stages * (bn + bm) * 128; }
constexpr int lds_split(int ni, int nj, int s) { return 4 * split_ring_bytes(ni, nj, s); }
constexpr int lds_direct(int waves) { return waves * 32 * 36 * 4; }
constexpr int kLdsGap = 4 * 64 * 4, kLdsRow = 16, kLdsNone = 0;
// ... of the bodies that group and chained kernels hold: the most a node of theirs asks for.
constexpr int kLdsLargestBody = std::max({lds_igemm(64, 64), lds_tile(128, 128, 2), lds_tile(64, 64, 3), lds_tile(128, 64, 2),
                                          lds_split(1, 1, 3), lds_split(2, 2, 2), lds_split(4, 2, 1), lds_split(4, 4, 1), lds_direct(4)});

// Operator timeline (tracing aid, off by default): while a buffer is set, thread 0 of every
// workgroup folds the 100 MHz device clock at its start and end into the operator's slot
// (two 64-bit words: earliest start, latest end).  It shows what a profiler cannot show
// without disturbing it: which operators of a replay really ran at the same time.
// The buffer travels as a kernel argument (null when off) and arrives with the others, so the
// clock is read only where somebody wants the stamp (a scalar clock read holds up every scalar
// load behind it).  Read from a device variable instead, the pointer put a dependent memory
// round trip in front of every workgroup's argument loads (GoogLeNet-like sequential graph 295
// -> 327 us with tracing off).
__device__ __forceinline__ unsigned long long op_trace_begin() { return (unsigned long long)wall_clock64(); }
// Only the operator's first workgroup reports a start and only its last eight (in dispatch
// order) an end: with every workgroup of a 2,000-workgroup operator updating the same two
// words the atomics serialised and doubled the time of a replay.
__device__ __forceinline__ void op_trace_end(unsigned long long *tr, int tag, unsigned long long t0, unsigned lin,
                                             unsigned total) {
  if (tr && threadIdx.x == 0) {
    if (lin == 0) atomicMin(tr + 2 * (size_t)tag, t0);
    if (lin + 8 >= total) atomicMax(tr + 2 * (size_t)tag + 1, (unsigned long long)wall_clock64());
  }
}
__device__ __forceinline__ unsigned launch_lin(const LaunchArgs &l) {
  return blockIdx.x + (unsigned)l.gx * (blockIdx.y + (unsigned)l.gy * blockIdx.z);
}
__device__ __forceinline__ unsigned launch_total(const LaunchArgs &l) { return (unsigned)l.gx * (unsigned)l.gy * (unsigned)l.gz; }

// The arguments of a kernel span up to five cache lines, and the compiler reads them where it
// needs them: one memory round trip after another at the head of every workgroup.  A contraction
// reads its whole record into scalar registers in one round; the other kernels read a word of
// every line first, which lets the later reads hit the scalar cache.
template <int BYTES> __device__ __forceinline__ void touch_arguments() {
  typedef const uint32_t __attribute__((address_space(4))) *CW;
  const CW w = (CW)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t a = w[0], b = w[(BYTES > 64 ? 64 : 0) / 4], c = w[(BYTES > 128 ? 128 : 0) / 4], d = w[(BYTES > 192 ? 192 : 0) / 4],
                 e = w[(BYTES - 4) / 4];
  asm volatile("" : : "s"(a), "s"(b), "s"(c), "s"(d), "s"(e));
}
template <typename Args> struct Hold {
  template <typename AR> static __device__ __forceinline__ void all(const AR &, const LaunchArgs &) {}
  static constexpr bool kOn = false;
};
template <> struct Hold<IgemmArgs> {
  template <typename AR> static __device__ __forceinline__ void all(const AR &a, const LaunchArgs &l) {
    asm volatile("" : : "s"(a.x), "s"(a.w), "s"(a.bias), "s"(a.y), "s"(a.n_extra), "s"(a.M), "s"(a.N), "s"(a.K), "s"(a.gather), "s"(a.H),
                 "s"(a.W), "s"(a.Cin), "s"(a.Wo), "s"(a.kh), "s"(a.kw), "s"(a.sh), "s"(a.sw), "s"(a.ph), "s"(a.pw), "s"(a.HoWo),
                 "s"((uint32_t)a.img_stride), "s"((uint32_t)a.lda), "s"((uint32_t)a.ldb), "s"(a.ldy), "s"(a.relu));
    asm volatile("" : : "s"(a.alpha), "s"(a.div_HoWo), "s"(a.div_Wo), "s"(a.div_Cin), "s"(a.div_kw), "s"(a.x_bytes), "s"(a.w_bytes),
                 "s"(a.div_gx), "s"(l.gx), "s"(l.gy));
  }
  static constexpr bool kOn = true;
};

// The operator's record, the launch's own arguments (KDEFT: and the element-wise operator that
// follows); nothing implicit, so that a kernel's argument segment is what is declared here: the
// grid of a launch (gridDim) would be read from 256 bytes that the runtime appends.
#define KBODY(ldsb, Args, call, extra)                                                           \
    __shared__ __attribute__((aligned(16))) unsigned char lds[(ldsb) > 0 ? (ldsb) : 16];         \
    if constexpr (!Hold<Args>::kOn) touch_arguments<sizeof(Args) + sizeof(LaunchArgs) + extra>();  \
    Hold<Args>::all(a, l);                                                                       \
    const Blk b = launch_blk(l);                                                                 \
    const unsigned long long t0 = l.trace ? op_trace_begin() : 0ull;                             \
    call;                                                                                        \
    op_trace_end(l.trace, l.tag, t0, launch_lin(l), launch_total(l));
#define KDEF(name, threads, ldsb, Args, call)                                                    \
  extern "C" __global__ void __launch_bounds__(threads) opara_k_##name(Args a, LaunchArgs l) {   \
    KBODY(ldsb, Args, call, 0)                                                                   \
  }
// second launch bound: wavefronts per SIMD the register allocation must leave room for
#define KDEF2(name, threads, waves_per_simd, ldsb, Args, call)                                   \
  extern "C" __global__ void __launch_bounds__(threads, waves_per_simd) opara_k_##name(Args a, LaunchArgs l) { \
    KBODY(ldsb, Args, call, 0)                                                                   \
  }
#define KDEFT(name, threads, waves_per_simd, ldsb, Args, call)                                   \
  extern "C" __global__ void __launch_bounds__(threads, waves_per_simd) opara_k_##name(Args a, LaunchArgs l, TailArgs tail) { \
    KBODY(ldsb, Args, call, sizeof(TailArgs))                                                    \
  }

KDEF2(igemm_f16_t128x64, 256, 2, lds_tile(128, 64, 2), IgemmArgs, (igemm_tile_body<half_t, 128, 64, 2, 2, 2, 0>(a, b, lds)))
KDEFT(igemm_f16_t128x64_tail, 256, 2, lds_tile(128, 64, 2), IgemmArgs, (igemm_tile_body<half_t, 128, 64, 2, 2, 2, 0>(a, b, lds, tail)))
KDEF2(igemm_f16_tile64x64, 256, 2, lds_tile(64, 64, 3), IgemmArgs, (igemm_tile_body<half_t, 64, 64, 2, 2, 3, 0>(a, b, lds)))
KDEFT(igemm_f16_tile64x64_tail, 256, 2, lds_tile(64, 64, 3), IgemmArgs, (igemm_tile_body<half_t, 64, 64, 2, 2, 3, 0>(a, b, lds, tail)))
KDEF2(igemm_f16_tile128x128, 256, 2, lds_tile(128, 128, 2), IgemmArgs, (igemm_tile_body<half_t, 128, 128, 2, 2, 2, 0>(a, b, lds)))
KDEFT(igemm_f16_tile128x128_tail, 256, 2, lds_tile(128, 128, 2), IgemmArgs, (igemm_tile_body<half_t, 128, 128, 2, 2, 2, 0>(a, b, lds, tail)))
KDEF2(igemm_f16_far128x128, 256, 2, lds_tile(128, 128, 2), IgemmArgs, (igemm_tile_body<half_t, 128, 128, 2, 2, 2, 0, true>(a, b, lds)))
KDEF2(igemm_f32_far128x128, 256, 2, lds_tile(128, 128, 2), IgemmArgs, (igemm_tile_body<float, 128, 128, 2, 2, 2, 0, true>(a, b, lds)))
KDEF(igemm_f16_t64x64, 256, lds_igemm(64, 64), IgemmArgs, (igemm_body<half_t, 64, 64, 2, 2, true, 0>(a, b, lds)))
KDEF(igemm_f16_direct4, 256, lds_direct(4), IgemmArgs, (igemm_direct_body<half_t, 4, 2, 0, 2, 2>(a, b, lds)))
KDEF2(igemm_f16_quad4, 256, 2, lds_split(2, 2, 2), IgemmArgs, (igemm_split_body<half_t, 2, 2, 2, 0>(a, b, lds)))
KDEFT(igemm_f16_quad4_tail, 256, 2, lds_split(2, 2, 2), IgemmArgs, (igemm_split_body<half_t, 2, 2, 2, 0>(a, b, lds, tail)))
KDEF2(igemm_f16_quad64x4, 256, 3, lds_split(4, 2, 1), IgemmArgs, (igemm_split_body<half_t, 4, 2, 1, 0>(a, b, lds)))
KDEFT(igemm_f16_quad64x4_tail, 256, 3, lds_split(4, 2, 1), IgemmArgs, (igemm_split_body<half_t, 4, 2, 1, 0>(a, b, lds, tail)))
KDEF2(igemm_f16_quad64x64, 256, 2, lds_split(4, 4, 1), IgemmArgs, (igemm_split_body<half_t, 4, 4, 1, 0>(a, b, lds)))
KDEFT(igemm_f16_quad64x64_tail, 256, 2, lds_split(4, 4, 1), IgemmArgs, (igemm_split_body<half_t, 4, 4, 1, 0>(a, b, lds, tail)))
KDEF(igemm_f16_t64x64_scalar, 256, lds_igemm(64, 64), IgemmArgs, (igemm_body<half_t, 64, 64, 2, 2, false, 0>(a, b, lds)))
KDEF2(igemm_f32_t128x64, 256, 2, lds_tile(128, 64, 2), IgemmArgs, (igemm_tile_body<float, 128, 64, 2, 2, 2, 0>(a, b, lds)))
KDEFT(igemm_f32_t128x64_tail, 256, 2, lds_tile(128, 64, 2), IgemmArgs, (igemm_tile_body<float, 128, 64, 2, 2, 2, 0>(a, b, lds, tail)))
KDEF2(igemm_f32_tile64x64, 256, 2, lds_tile(64, 64, 3), IgemmArgs, (igemm_tile_body<float, 64, 64, 2, 2, 3, 0>(a, b, lds)))
KDEFT(igemm_f32_tile64x64_tail, 256, 2, lds_tile(64, 64, 3), IgemmArgs, (igemm_tile_body<float, 64, 64, 2, 2, 3, 0>(a, b, lds, tail)))
KDEF2(igemm_f32_tile128x128, 256, 2, lds_tile(128, 128, 2), IgemmArgs, (igemm_tile_body<float, 128, 128, 2, 2, 2, 0>(a, b, lds)))
KDEFT(igemm_f32_tile128x128_tail, 256, 2, lds_tile(128, 128, 2), IgemmArgs, (igemm_tile_body<float, 128, 128, 2, 2, 2, 0>(a, b, lds, tail)))
KDEF(igemm_f32_t64x64, 256, lds_igemm(64, 64), IgemmArgs, (igemm_body<float, 64, 64, 2, 2, true, 0>(a, b, lds)))
KDEF(igemm_f32_direct4, 256, lds_direct(4), IgemmArgs, (igemm_direct_body<float, 4, 2, 0, 2, 2>(a, b, lds)))
KDEF2(igemm_f32_quad4, 256, 2, lds_split(2, 2, 2), IgemmArgs, (igemm_split_body<float, 2, 2, 2, 0>(a, b, lds)))
KDEFT(igemm_f32_quad4_tail, 256, 2, lds_split(2, 2, 2), IgemmArgs, (igemm_split_body<float, 2, 2, 2, 0>(a, b, lds, tail)))
KDEF2(igemm_f32_quad64x4, 256, 3, lds_split(4, 2, 1), IgemmArgs, (igemm_split_body<float, 4, 2, 1, 0>(a, b, lds)))
KDEFT(igemm_f32_quad64x4_tail, 256, 3, lds_split(4, 2, 1), IgemmArgs, (igemm_split_body<float, 4, 2, 1, 0>(a, b, lds, tail)))
KDEF2(igemm_f32_quad64x64, 256, 2, lds_split(4, 4, 1), IgemmArgs, (igemm_split_body<float, 4, 4, 1, 0>(a, b, lds)))
KDEFT(igemm_f32_quad64x64_tail, 256, 2, lds_split(4, 4, 1), IgemmArgs, (igemm_split_body<float, 4, 4, 1, 0>(a, b, lds, tail)))
KDEF(igemm_f32_t64x64_scalar, 256, lds_igemm(64, 64), IgemmArgs, (igemm_body<float, 64, 64, 2, 2, false, 0>(a, b, lds)))
KDEF(gemv_f16, 256, kLdsNone, IgemmArgs, (gemv_body<half_t, 0>(a, b, lds)))
KDEF(gemv_f32, 256, kLdsNone, IgemmArgs, (gemv_body<float, 0>(a, b, lds)))
KDEF(pool_f16_vec, 256, kLdsNone, PoolArgs, (pool_body<half_t, 8, 0>(a, b, lds)))
KDEF(pool_f16_scalar, 256, kLdsNone, PoolArgs, (pool_body<half_t, 1, 0>(a, b, lds)))
KDEF(pool_f32_vec, 256, kLdsNone, PoolArgs, (pool_body<float, 4, 0>(a, b, lds)))
KDEF(pool_f32_scalar, 256, kLdsNone, PoolArgs, (pool_body<float, 1, 0>(a, b, lds)))
KDEF(gap_f16, 256, kLdsGap, GapArgs, (gap_body<half_t, 0>(a, b, lds)))
KDEF(gap_f32, 256, kLdsGap, GapArgs, (gap_body<float, 0>(a, b, lds)))
KDEF(layernorm_f16_wave, 256, kLdsRow, RowArgs, (row_cached_body<half_t, true, 64, 2, 0>(a, b, lds)))
KDEF(layernorm_f16_block, 256, kLdsRow, RowArgs, (row_cached_body<half_t, true, 256, kRowCacheChunks, 0>(a, b, lds)))
KDEF(layernorm_f16_generic, 256, kLdsRow, RowArgs, (row_generic_body<half_t, true, 0>(a, b, lds)))
KDEF(layernorm_f32_wave, 256, kLdsRow, RowArgs, (row_cached_body<float, true, 64, 2, 0>(a, b, lds)))
KDEF(layernorm_f32_block, 256, kLdsRow, RowArgs, (row_cached_body<float, true, 256, kRowCacheChunks, 0>(a, b, lds)))
KDEF(layernorm_f32_generic, 256, kLdsRow, RowArgs, (row_generic_body<float, true, 0>(a, b, lds)))
KDEF(softmax_f16_wave, 256, kLdsRow, RowArgs, (row_cached_body<half_t, false, 64, 2, 0>(a, b, lds)))
KDEF(softmax_f16_block, 256, kLdsRow, RowArgs, (row_cached_body<half_t, false, 256, kRowCacheChunks, 0>(a, b, lds)))
KDEF(softmax_f16_generic, 256, kLdsRow, RowArgs, (row_generic_body<half_t, false, 0>(a, b, lds)))
KDEF(softmax_f32_wave, 256, kLdsRow, RowArgs, (row_cached_body<float, false, 64, 2, 0>(a, b, lds)))
KDEF(softmax_f32_block, 256, kLdsRow, RowArgs, (row_cached_body<float, false, 256, kRowCacheChunks, 0>(a, b, lds)))
KDEF(softmax_f32_generic, 256, kLdsRow, RowArgs, (row_generic_body<float, false, 0>(a, b, lds)))
KDEF(elt_f16_vec, 256, kLdsNone, EltArgs, (elt_body<half_t, 8, 0>(a, b, lds)))
KDEF(elt_f16_scalar, 256, kLdsNone, EltArgs, (elt_body<half_t, 1, 0>(a, b, lds)))
KDEF(elt_f32_vec, 256, kLdsNone, EltArgs, (elt_body<float, 4, 0>(a, b, lds)))
KDEF(elt_f32_scalar, 256, kLdsNone, EltArgs, (elt_body<float, 1, 0>(a, b, lds)))
KDEF(concat_f16_vec, 256, kLdsNone, ConcatArgs, (concat_body<half_t, 8, 0>(a, b, lds)))
KDEF(concat_f16_scalar, 256, kLdsNone, ConcatArgs, (concat_body<half_t, 1, 0>(a, b, lds)))
KDEF(concat_f32_vec, 256, kLdsNone, ConcatArgs, (concat_body<float, 4, 0>(a, b, lds)))
KDEF(concat_f32_scalar, 256, kLdsNone, ConcatArgs, (concat_body<float, 1, 0>(a, b, lds)))
// 16 x 16 output tiles: four times the workgroups of the 32 x 32 forms, half the operand bytes per workgroup
KDEF(igemm_f16_direct4s, 256, lds_direct(4), IgemmArgs, (igemm_direct_body<half_t, 4, 2, 0, 1, 1>(a, b, lds)))
KDEF2(igemm_f16_quad4s, 256, 3, lds_split(1, 1, 3), IgemmArgs, (igemm_split_body<half_t, 1, 1, 3, 0>(a, b, lds)))
KDEFT(igemm_f16_quad4s_tail, 256, 3, lds_split(1, 1, 3), IgemmArgs, (igemm_split_body<half_t, 1, 1, 3, 0>(a, b, lds, tail)))
KDEF(igemm_f32_direct4s, 256, lds_direct(4), IgemmArgs, (igemm_direct_body<float, 4, 2, 0, 1, 1>(a, b, lds)))
KDEF2(igemm_f32_quad4s, 256, 3, lds_split(1, 1, 3), IgemmArgs, (igemm_split_body<float, 1, 1, 3, 0>(a, b, lds)))
KDEFT(igemm_f32_quad4s_tail, 256, 3, lds_split(1, 1, 3), IgemmArgs, (igemm_split_body<float, 1, 1, 3, 0>(a, b, lds, tail)))

KDEF2(attention_f16, 256, 2, kLdsAttention, AttnArgs, (attention_body(a, b, lds)))

// The 256-thread bodies by the vector registers they need (see the group kernels below):
// X(kernel name, argument record, body call); T / tn: element type, C: access policy.
#define STREAM_BODIES(X, T, VE, tn, C)                                                                        \
  X(gemv_##tn, IgemmArgs, (gemv_body<T, C>(a, b, lds)))                                                       \
  X(pool_##tn##_vec, PoolArgs, (pool_body<T, VE, C>(a, b, lds)))                                              \
  X(pool_##tn##_scalar, PoolArgs, (pool_body<T, 1, C>(a, b, lds)))                                            \
  X(gap_##tn, GapArgs, (gap_body<T, C>(a, b, lds)))                                                           \
  X(layernorm_##tn##_wave, RowArgs, (row_cached_body<T, true, 64, 2, C>(a, b, lds)))                          \
  X(layernorm_##tn##_block, RowArgs, (row_cached_body<T, true, 256, kRowCacheChunks, C>(a, b, lds)))          \
  X(layernorm_##tn##_generic, RowArgs, (row_generic_body<T, true, C>(a, b, lds)))                             \
  X(softmax_##tn##_wave, RowArgs, (row_cached_body<T, false, 64, 2, C>(a, b, lds)))                           \
  X(softmax_##tn##_block, RowArgs, (row_cached_body<T, false, 256, kRowCacheChunks, C>(a, b, lds)))           \
  X(softmax_##tn##_generic, RowArgs, (row_generic_body<T, false, C>(a, b, lds)))                              \
  X(elt_##tn##_vec, EltArgs, (elt_body<T, VE, C>(a, b, lds)))                                                 \
  X(elt_##tn##_scalar, EltArgs, (elt_body<T, 1, C>(a, b, lds)))                                               \
  X(concat_##tn##_vec, ConcatArgs, (concat_body<T, VE, C>(a, b, lds)))                                        \
  X(concat_##tn##_scalar, ConcatArgs, (concat_body<T, 1, C>(a, b, lds)))
#define LIGHT_BODIES(X, T, tn, C)                                                                             \
  X(igemm_##tn##_t64x64, IgemmArgs, (igemm_body<T, 64, 64, 2, 2, true, C>(a, b, lds)))                        \
  X(igemm_##tn##_t64x64_scalar, IgemmArgs, (igemm_body<T, 64, 64, 2, 2, false, C>(a, b, lds)))                \
  X(igemm_##tn##_direct4, IgemmArgs, (igemm_direct_body<T, 4, 2, C, 2, 2>(a, b, lds)))                        \
  X(igemm_##tn##_direct4s, IgemmArgs, (igemm_direct_body<T, 4, 2, C, 1, 1>(a, b, lds)))                       \
  X(igemm_##tn##_quad4s, IgemmArgs, (igemm_split_body<T, 1, 1, 3, C>(a, b, lds)))                             \
  X(igemm_##tn##_quad4, IgemmArgs, (igemm_split_body<T, 2, 2, 2, C>(a, b, lds)))
#define HEAVY_BODIES(X, T, tn, C)                                                                             \
  X(igemm_##tn##_quad64x4, IgemmArgs, (igemm_split_body<T, 4, 2, 1, C>(a, b, lds)))                           \
  X(igemm_##tn##_quad64x64, IgemmArgs, (igemm_split_body<T, 4, 4, 1, C>(a, b, lds)))                          \
  X(igemm_##tn##_tile64x64, IgemmArgs, (igemm_tile_body<T, 64, 64, 2, 2, 3, C>(a, b, lds)))                   \
  X(igemm_##tn##_t128x64, IgemmArgs, (igemm_tile_body<T, 128, 64, 2, 2, 2, C>(a, b, lds)))                    \
  X(igemm_##tn##_tile128x128, IgemmArgs, (igemm_tile_body<T, 128, 128, 2, 2, 2, C>(a, b, lds)))
// heavy too, but not in the chained kernel (where it costs the other bodies 1 %: BERT-like 1081 -> 1093 us)
#define FAR_BODIES(X, T, tn, C)                                                                               \
  X(igemm_##tn##_far128x128, IgemmArgs, (igemm_tile_body<T, 128, 128, 2, 2, 2, C, true>(a, b, lds)))

// ---------------------------------------------------------------------------------
// Persistent executor.  One launch runs the whole DAG: each workgroup repeatedly takes
// the next ticket, finds the operator and tile it denotes, waits until that operator's
// predecessors have completed all their tiles, runs the tile with the operator's own
// body, and publishes the completion.  Tickets follow the launch queue, which is a
// topological order, so the owner of the lowest unfinished ticket never waits for a
// ticket nobody holds: the launch drains whatever number of workgroups is resident.
// Every wait is bounded; a wait that runs out sets the sticky error word and all
// workgroups leave.  The last workgroup to leave clears the counters for the next launch.
// ---------------------------------------------------------------------------------
template <typename A> __device__ __forceinline__ A load_uniform(const void *p) {
  // Records are written once before the first launch and never by a kernel: read them
  // through the constant address space so they arrive in scalar registers like
  // ordinary kernel arguments.
  typedef const uint32_t __attribute__((address_space(4))) *CP;
  CP w = (CP)(uintptr_t)p;
  union { A a; uint32_t w[sizeof(A) / 4]; } u;
  static_assert(sizeof(A) % 4 == 0, "record size");
#pragma unroll
  for (unsigned i = 0; i < sizeof(A) / 4; ++i) u.w[i] = w[i];
  return u.a;
}

// Loads inside the persistent kernel are plain: each work item starts with one cache
// invalidate (acquire at device scope).  (Device-coherent loads instead cost 5-10 % more
// latency: every operand re-read goes past the L2.)
// TILED: the kernel holds the 128 x 64 tile for heavy contractions as well.  Its scalar state makes the
// compiler spill in the loop around every body, so that DAGs without such a contraction run without
// it (us: BERT-like 1171 -> 1154, Inception-v3-like 458 -> 453, NASNet-like 157 -> 154).
template <bool F16, bool TILED>
__device__ __forceinline__ void persist_run(int kernel, const PersistOp *r, const Blk &b, unsigned char *lds) {
#define PCASE(name, Args, call)                               \
  case K_##name: {                                            \
    typedef const Args __attribute__((address_space(4))) CA;  \
    CA &a = *(CA *)(uintptr_t)&r->args;                       \
    call;                                                     \
  } break;
#define PERSIST_BODIES(T, VE, tn)                                                                             \
  PCASE(igemm_##tn##_t64x64, IgemmArgs, (igemm_body<T, 64, 64, 2, 2, true, kCohStore>(a, b, lds)))            \
  PCASE(igemm_##tn##_direct4, IgemmArgs, (igemm_direct_body<T, 4, 2, kCohStore, 2, 2>(a, b, lds)))            \
  PCASE(igemm_##tn##_t64x64_scalar, IgemmArgs, (igemm_body<T, 64, 64, 2, 2, false, kCohStore>(a, b, lds)))    \
  STREAM_BODIES(PCASE, T, VE, tn, kCohStore)
  if constexpr (F16) {
    switch (kernel) {
      PERSIST_BODIES(half_t, 8, f16)
      default:
        if constexpr (TILED) {
          switch (kernel) {
            PCASE(igemm_f16_t128x64, IgemmArgs, (igemm_tile_body<half_t, 128, 64, 2, 2, 2, kCohStore>(a, b, lds)))
            default: break;
          }
        }
        break;
    }
  } else {
    switch (kernel) {
      PERSIST_BODIES(float, 4, f32)
      default:
        if constexpr (TILED) {
          switch (kernel) {
            PCASE(igemm_f32_t128x64, IgemmArgs, (igemm_tile_body<float, 128, 64, 2, 2, 2, kCohStore>(a, b, lds)))
            default: break;
          }
        }
        break;
    }
  }
#undef PERSIST_BODIES
#undef PCASE
}

// Thread 0 only: wait until every predecessor of the operator at queue position `pos`
// has raised its flag for this launch.  Each workgroup polls its own copy of a flag
// (hundreds of workgroups polling one address queue up behind each other, and the
// counter updates behind them).  False: the wait ran out, or another workgroup's did.
__device__ __forceinline__ bool persist_wait(const PersistArgs &pa, const PersistPredsLds *pl, int pos, uint32_t epoch,
                                             uint32_t limit) {
  const int np = pl->n;
  const uint32_t copy = (blockIdx.x % kPersistReplicas) * kPersistFlagStride;
  uint32_t spins = 0;
  for (int j = 0; j < np; ++j) {
    const uint32_t *f = pa.flags + (size_t)pl->pos[j] * (kPersistReplicas * kPersistFlagStride) + copy;
    while (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != epoch) {
      ++spins;
      if (spins > limit) {
        __hip_atomic_store(&pa.hdr->error, (uint32_t)pos + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
      }
      if ((spins & 31u) == 0 && __hip_atomic_load(&pa.hdr->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
        return false;
      __builtin_amdgcn_s_sleep(1);
    }
  }
  return true;
}

// Thread 0 only, after the workgroup's stores are complete: count the finished tiles of
// the operator at `pos`; whoever counts the last tile clears the counter for the next
// launch and raises every copy of the operator's flag.
__device__ __forceinline__ void persist_publish(const PersistArgs &pa, const PersistPredsLds *preds, int pos, uint32_t count,
                                                uint32_t epoch) {
  uint32_t *d = pa.done + (size_t)pos * kPersistCounterStride;
  const uint32_t before = __hip_atomic_fetch_add(d, count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (before + count == (uint32_t)preds[pos].tiles) {
    __hip_atomic_store(d, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t *f = pa.flags + (size_t)pos * (kPersistReplicas * kPersistFlagStride);
#pragma unroll
    for (int r = 0; r < kPersistReplicas; ++r)
      __hip_atomic_store(f + r * kPersistFlagStride, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Queue position of work item `item` (uniform; table in workgroup memory, begin[n] = total).
__device__ __forceinline__ int persist_find(const int32_t *begin, int n, uint32_t item) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((uint32_t)begin[mid] <= item) lo = mid; else hi = mid;
  }
  return lo;
}

// Work items are dealt round-robin: workgroup g runs items g, g + G, g + 2G, ... of the
// launch queue, each after its operator's predecessors are complete.  The queue is a
// topological order and every workgroup of the launch is resident (the host sizes G to
// the occupancy), so the owner of the lowest unfinished item is always able to run it.
//
// Every activation access inside the bodies is device-coherent (see ldg/stg), so an item
// is published by waiting for the workgroup's stores and then bumping the operator's
// counter with relaxed atomics; a consumer that has read the full count may read the data.
//
// Each iteration has exactly ONE thread-0-only region (publish the previous item, await
// the predecessors of this one), placed before the first of its two barriers.  With a
// second such region after the last barrier the compiler threads thread 0 from the end of
// one iteration straight into the next; the other lanes of its wavefront then reach the
// barrier on their own, the wavefront arrives twice and the barrier count of the
// workgroup no longer matches.
template <bool F16, bool TILED>
__device__ __forceinline__ void persist_body(const PersistArgs &pa) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_lds[];
  unsigned char *lds = dyn_lds;                                  // kPersistBodyLds bytes for the bodies
  int32_t *ctl = (int32_t *)(dyn_lds + kPersistBodyLds);         // [4] abort flag, -, last-out flag
  int32_t *begin = ctl + 4;                                      // [n + 1]
  const PersistPredsLds *preds = (const PersistPredsLds *)(begin + pa.n + 1);   // [n]
  const int tid = threadIdx.x;
  for (int i = tid; i <= pa.n; i += 256) begin[i] = pa.item_begin[i];
  {
    const uint32_t *src = (const uint32_t *)pa.preds;
    uint32_t *dst = (uint32_t *)(begin + pa.n + 1);
    const int words = pa.n * (int)(sizeof(PersistPredsLds) / 4);
    for (int i = tid; i < words; i += 256) dst[i] = src[i];
  }
  if (tid == 0) ctl[0] = 0;
  // Optional timeline: four 64-bit words per work item (constant 100 MHz clock): lookup
  // started, predecessors complete, body finished, (queue position << 32 | workgroup).
  uint64_t *trace = nullptr;
  uint32_t limit = 0, epoch = 0;
  uint64_t t_begin = 0, t_ready = 0;
  if (tid == 0) {
    trace = (uint64_t *)__hip_atomic_load(&pa.hdr->trace, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    limit = __hip_atomic_load(&pa.hdr->spin_limit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    epoch = __hip_atomic_load(&pa.hdr->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  int prev = -1;
  uint32_t prev_count = 0, sink = 0;
  for (uint32_t item = blockIdx.x; item < (uint32_t)pa.total; item += gridDim.x) {
    const int pos = __builtin_amdgcn_readfirstlane(persist_find(begin, pa.n, item));
    // A work item is `chunk` consecutive tiles of one operator (operators with more tiles
    // than the launch has workgroups: one acquire, one record, one publication for the lot).
    // Operators start at multiples of kPersistItemAlign in the item space; the items that
    // pad an operator out denote no tile.
    const int chunk = preds[pos].chunk;
    const int tile0 = (int)(item - (uint32_t)begin[pos]) * chunk;
    const int op_tiles = preds[pos].tiles;
    const bool padding = tile0 >= op_tiles;
    const int ntiles = padding ? 0 : min(chunk, op_tiles - tile0);
    if (tid == 0) {
      if (prev >= 0) {
        persist_publish(pa, preds, prev, prev_count, epoch);
        if (trace) {
          uint64_t *rec = trace + 4 * (uint64_t)(item - gridDim.x);
          const uint64_t t_end = wall_clock64();
          rec[0] = t_begin; rec[1] = t_ready; rec[2] = t_end;
          rec[3] = ((uint64_t)(uint32_t)prev << 32) | blockIdx.x;
        }
      }
      if (trace) t_begin = wall_clock64();
      if (!padding && !persist_wait(pa, preds + pos, pos, epoch, limit)) ctl[0] = 1;
      if (trace) t_ready = wall_clock64();
    }
    if (tid < 64)                                                // one wavefront invalidates the caches this
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");         // workgroup reads through (L1 of the CU, L2 of the XCD)
    __syncthreads();                                             // predecessors complete (or abort)
    if (ctl[0]) { prev = -1; break; }
    if (padding) { prev = -1; continue; }
    const PersistOp *r = pa.rec + pos;
    const int4 hd = load_uniform<int4>(r);                       // kernel, gx, gy, gz
    Blk b;
    b.gx = hd.y; b.gy = hd.z;
    // With the workgroup count and every operator's first item multiples of the XCD count,
    // tile t of an unchunked operator runs on XCD t % 8 exactly as in an ordinary launch:
    // the same remap applies.  A chunk keeps consecutive tiles (neighbours that share
    // operand rows) in one workgroup instead.
    b.remap = chunk == 1 && (gridDim.x % kPersistItemAlign) == 0;
    for (int k = 0; k < ntiles; ++k) {
      const int tile = tile0 + k;
      b.x = tile % hd.y;
      const int rest = tile / hd.y;
      b.y = rest % hd.z;
      b.z = rest / hd.z;
      b.lin = b.y * hd.y + b.x;
      if (k > 0) __syncthreads();                                // the previous tile is done with workgroup memory
      persist_run<F16, TILED>(hd.x, r, b, lds);
    }
    // While the stores drain: touch the next item's record so that its argument loads find
    // it in the scalar cache.  The values only feed a sink that is tested after the loop.
    {
      const uint32_t nitem = item + gridDim.x;
      const int npos = nitem < (uint32_t)pa.total ? persist_find(begin, pa.n, nitem) : pos;
      const unsigned char *nr = (const unsigned char *)(pa.rec + __builtin_amdgcn_readfirstlane(npos));
      const uint32_t p0 = load_uniform<uint32_t>(nr), p1 = load_uniform<uint32_t>(nr + 64);
      const uint32_t p2 = load_uniform<uint32_t>(nr + 128), p3 = load_uniform<uint32_t>(nr + 192);
      sink += (p0 ^ p1) + (p2 ^ p3);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                          // vmcnt(0): this wavefront's stores are complete
    __syncthreads();                                             // ... for every wavefront, and ctl has been read
    prev = pos;
    prev_count = (uint32_t)ntiles;
  }
  // Leave: publish the last item; the last workgroup out clears the counters (nobody is
  // left to read them) and advances the launch number.
  if (tid == 0) {
    if (prev >= 0) {
      persist_publish(pa, preds, prev, prev_count, epoch);
      if (trace) {
        // the loop has advanced `item` past the end: the last item of this workgroup is the
        // largest g + k*G below total
        const uint32_t last = blockIdx.x + ((uint32_t)pa.total - 1u - blockIdx.x) / gridDim.x * gridDim.x;
        uint64_t *rec = trace + 4 * (uint64_t)last;
        rec[0] = t_begin; rec[1] = t_ready; rec[2] = wall_clock64();
        rec[3] = ((uint64_t)(uint32_t)prev << 32) | blockIdx.x;
      }
    }
    if (sink == 0x9e3779b9u) pa.hdr->reserved0 = sink;           // keeps the record touches alive
    const uint32_t e = __hip_atomic_fetch_add(&pa.hdr->exited, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ctl[2] = (e == gridDim.x - 1) ? 1 : 0;
  }
  __syncthreads();
  if (ctl[2]) {
    // Counters of operators that did not complete (abandoned launch) would poison the
    // next one; after a clean launch they are all zero already.
    for (int i = tid; i < pa.n; i += 256) pa.done[(size_t)i * kPersistCounterStride] = 0u;
    if (tid == 0) {
      pa.hdr->exited = 0u;
      pa.hdr->epoch = epoch + 1u;
    }
  }
}

extern "C" __global__ void __launch_bounds__(256, 2) opara_k_persist_f16(PersistArgs pa) { persist_body<true, false>(pa); }
extern "C" __global__ void __launch_bounds__(256, 2) opara_k_persist_f32(PersistArgs pa) { persist_body<false, false>(pa); }
extern "C" __global__ void __launch_bounds__(256, 2) opara_k_persist_f16_tiled(PersistArgs pa) { persist_body<true, true>(pa); }
extern "C" __global__ void __launch_bounds__(256, 2) opara_k_persist_f32_tiled(PersistArgs pa) { persist_body<false, true>(pa); }

// ---------------------------------------------------------------------------------
// Group kernel (fused executor): one launch runs several mutually independent operators.
// A workgroup finds its operator from the block ranges in the argument record, rebuilds
// its position in that operator's own grid and runs the operator's ordinary body on the
// operator's arguments, which it reads from the kernel-argument segment like any kernel
// does.  No flags, no coherent accesses: kernel boundaries order the groups.  Three flavours
// per element type, by the registers their bodies need: "stream" (at most 64: pooling,
// row-wise, element-wise, concatenation, matrix-vector; eight wavefronts per SIMD stay
// resident, which streaming wants), "light" (at most 128: those plus the register-staged, the
// fragment-loading and the 16 x 16 and 32 x 32 LDS-fed contractions; four per SIMD), "heavy" (all
// 256-thread bodies; two).  Every workgroup of a group has the workgroup memory of its largest
// member: beside a 16 x 16 LDS-fed contraction (48 KB) three of them share a CU, beside a 32 x 32
// one (64 KB) two, whatever the registers would allow.
// ---------------------------------------------------------------------------------
template <bool F16, int FLAVOR, bool TRACE>
__device__ __forceinline__ void group_body() {
  // The record is the kernel's only argument and therefore starts the kernel-argument
  // segment.  It is read in place through the segment pointer: indexing the by-value
  // parameter with a run-time operator number would make the compiler copy all of it into
  // private memory first.
  typedef const GroupArgs __attribute__((address_space(4))) CGA;
  CGA &ga = *(CGA *)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_lds[];
  const int blk = (int)blockIdx.x;
  // The member this block belongs to: all sixteen range ends arrive with one 64-byte load
  // (unused entries hold INT32_MAX), the member is the number of ends at or below the block.
  // Range ends, shape and arguments all come from the one record in memory.  Taking the ends
  // from registers that the hardware fills ahead of the workgroup (preloaded arguments) saves a
  // round trip, 0.45 us a node, but then two sources have to agree before a store is in bounds.
  int i = 0;
#pragma unroll
  for (int j = 0; j < kGroupMaxOps - 1; ++j) i += blk >= ga.block_end[j] ? 1 : 0;
  i = __builtin_amdgcn_readfirstlane(i);
  // The member's launch shape and, in the same round, a word of every cache line of its argument
  // record, so that the body's own argument loads (which the compiler issues only behind the
  // switch below) find it in the scalar cache instead of paying another memory round trip.
  typedef const uint32_t __attribute__((address_space(4))) *CW;
  const CW rec = (CW)&ga.args[i];
  typedef const GroupMeta __attribute__((address_space(4))) CM;
  CM &me = ga.meta[i];
  asm volatile("" : : "s"(me.kernel), "s"(me.gx), "s"(me.gy), "s"(me.tiles), "s"(me.block_begin), "s"(me.div_gx), "s"(me.gz),
               "s"(rec[0]), "s"(rec[16]), "s"(rec[32]), "s"(rec[sizeof(KernelArgs) / 4 - 1]));
  const int tile = blk - me.block_begin;
  if ((uint32_t)tile >= (uint32_t)me.tiles) return;                // padding of the operator's range
  Blk b;
  b.gx = me.gx; b.gy = me.gy;
  b.remap = true;
  b.z = 0;
  b.lin = tile;
  if (me.gz > 1) {
    b.z = tile / (b.gx * b.gy);
    b.lin = tile - b.z * (b.gx * b.gy);
  }
  b.y = (int)fast_div((uint32_t)b.lin, (uint32_t)b.gx, me.div_gx);
  b.x = b.lin - b.y * b.gx;
  unsigned char *lds = dyn_lds;
  // traced instances are separate kernels: even an unused clock read at the start of this
  // kernel's chain of dependent scalar loads cost every group node 0.4 us
  const int tag = TRACE ? me.tag : 0;
  const unsigned long long t0 = TRACE ? op_trace_begin() : 0ull;
#define GCASE(name, Args, call)                               \
  case K_##name: {                                            \
    typedef const Args __attribute__((address_space(4))) CA;  \
    CA &a = *(CA *)&ga.args[i];                               \
    call;                                                     \
  } break;
  if constexpr (F16) {
    switch (me.kernel) {
      STREAM_BODIES(GCASE, half_t, 8, f16, 0)
      default:
        if constexpr (FLAVOR >= 1) {
          switch (me.kernel) {
            LIGHT_BODIES(GCASE, half_t, f16, 0)
            default:
              if constexpr (FLAVOR >= 2) {
                switch (me.kernel) {
                  HEAVY_BODIES(GCASE, half_t, f16, 0)
                  FAR_BODIES(GCASE, half_t, f16, 0)
                  default: break;
                }
              }
              break;
          }
        }
        break;
    }
  } else {
    switch (me.kernel) {
      STREAM_BODIES(GCASE, float, 4, f32, 0)
      default:
        if constexpr (FLAVOR >= 1) {
          switch (me.kernel) {
            LIGHT_BODIES(GCASE, float, f32, 0)
            default:
              if constexpr (FLAVOR >= 2) {
                switch (me.kernel) {
                  HEAVY_BODIES(GCASE, float, f32, 0)
                  FAR_BODIES(GCASE, float, f32, 0)
                  default: break;
                }
              }
              break;
          }
        }
        break;
    }
  }
#undef GCASE
  if constexpr (TRACE) op_trace_end(ga.trace, tag, t0, (unsigned)tile, (unsigned)me.tiles);
}

#define GROUPK2(name, waves, F16, FLAVOR, TRACE) \
  extern "C" __global__ void __launch_bounds__(256, waves) opara_k_group_##name(GroupArgs) { group_body<F16, FLAVOR, TRACE>(); }
#define GROUPK(name, waves, F16, FLAVOR) GROUPK2(name, waves, F16, FLAVOR, false) GROUPK2(name##_traced, waves, F16, FLAVOR, true)
GROUPK(f16_stream, 8, true, 0)
GROUPK(f16_light, 4, true, 1)
GROUPK(f16_heavy, 2, true, 2)
GROUPK(f32_stream, 8, false, 0)
GROUPK(f32_light, 4, false, 1)
GROUPK(f32_heavy, 2, false, 2)
#undef GROUPK

// ---------------------------------------------------------------------------------
// Chained executor: every workgroup runs one tile of one operator behind a wait for the
// operator's predecessors (see ChainArgs).  Same hand-off as the persistent kernel (results
// through device-coherent stores, completion counters and replicated flags, one cache
// invalidate per workgroup), but no loop: a body is straight-line code behind the wait, so
// nothing is hoisted across bodies, the LDS-fed contractions can be held, and the
// launch does not depend on all its workgroups being resident at once.
// ---------------------------------------------------------------------------------
template <bool F16, bool LIGHT>
__device__ __forceinline__ void chain_body(const ChainArgs &pa) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_lds[];
  __shared__ int32_t ctl[2];
  typedef const int32_t __attribute__((address_space(4))) *CI;
  const int blk = (int)blockIdx.x;
  const int pos = __builtin_amdgcn_readfirstlane(((CI)(uintptr_t)pa.block_op)[blk]);
  if (pos < 0) return;                                            // padding of an operator's block range
  typedef const ChainRec __attribute__((address_space(4))) CR;
  CR &r = *(CR *)(uintptr_t)(pa.rec + pos);
  const int tid = threadIdx.x;
  uint64_t *trace = nullptr;
  uint64_t t_begin = 0, t_ready = 0;
  uint32_t epoch = 0;
  if (tid == 0) {
    trace = (uint64_t *)__hip_atomic_load(&pa.hdr->trace, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (trace) t_begin = wall_clock64();
    const uint32_t limit = __hip_atomic_load(&pa.hdr->spin_limit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    epoch = __hip_atomic_load(&pa.hdr->epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint32_t copy = ((uint32_t)blk % kPersistReplicas) * kPersistFlagStride;
    const int np = r.n_preds;
    uint32_t spins = 0;
    int ok = 1;
    for (int j = 0; j < np && ok; ++j) {
      const uint32_t *f = pa.flags + (size_t)r.preds[j] * (kPersistReplicas * kPersistFlagStride) + copy;
      while (__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != epoch) {
        if (++spins > limit) {
          __hip_atomic_store(&pa.hdr->error, (uint32_t)pos + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ok = 0;
          break;
        }
        if ((spins & 31u) == 0 && __hip_atomic_load(&pa.hdr->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    ctl[0] = ok;
    if (trace) t_ready = wall_clock64();
  }
  if (tid < 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // after the wait (thread 0 is in this wavefront)
  __syncthreads();
  if (!ctl[0]) return;                                            // a wait ran out somewhere: leave, publish nothing
  Blk b;
  b.gx = r.gx; b.gy = r.gy;
  b.remap = true;
  const int tile = blk - r.begin;
  b.x = tile % b.gx;
  const int rest = tile / b.gx;
  b.y = rest % b.gy;
  b.z = rest / b.gy;
  b.lin = b.y * b.gx + b.x;
  unsigned char *lds = dyn_lds;
#define CCASE(name, Args, call)                               \
  case K_##name: {                                            \
    typedef const Args __attribute__((address_space(4))) CA;  \
    CA &a = *(CA *)&r.args;                                   \
    call;                                                     \
  } break;
  if constexpr (F16) {
    switch (r.kernel) {
      STREAM_BODIES(CCASE, half_t, 8, f16, kCohStore)
      default:
        if constexpr (true) {
          switch (r.kernel) {
            LIGHT_BODIES(CCASE, half_t, f16, kCohStore)
            default:
              if constexpr (!LIGHT) {
                switch (r.kernel) {
                  HEAVY_BODIES(CCASE, half_t, f16, kCohStore)
                  default: break;
                }
              }
              break;
          }
        }
        break;
    }
  } else {
    switch (r.kernel) {
      STREAM_BODIES(CCASE, float, 4, f32, kCohStore)
      default:
        if constexpr (true) {
          switch (r.kernel) {
            LIGHT_BODIES(CCASE, float, f32, kCohStore)
            default:
              if constexpr (!LIGHT) {
                switch (r.kernel) {
                  HEAVY_BODIES(CCASE, float, f32, kCohStore)
                  default: break;
                }
              }
              break;
          }
        }
        break;
    }
  }
#undef CCASE
  __builtin_amdgcn_s_waitcnt(0x0F70);                            // vmcnt(0): this wavefront's stores are complete
  __syncthreads();                                               // ... for every wavefront of the workgroup
  if (tid == 0) {
    uint32_t *d = pa.done + (size_t)pos * kPersistCounterStride;
    const uint32_t before = __hip_atomic_fetch_add(d, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (before + 1u == (uint32_t)r.tiles) {                      // the operator's last tile: raise its flags
      __hip_atomic_store(d, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      uint32_t *f = pa.flags + (size_t)pos * (kPersistReplicas * kPersistFlagStride);
#pragma unroll
      for (int q = 0; q < kPersistReplicas; ++q)
        __hip_atomic_store(f + q * kPersistFlagStride, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // the last operator to complete advances the launch number for the next replay
      const uint32_t ops = __hip_atomic_fetch_add(&pa.hdr->exited, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (ops + 1u == (uint32_t)pa.n) {
        __hip_atomic_store(&pa.hdr->exited, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&pa.hdr->epoch, epoch + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
    if (trace) {
      uint64_t *rec = trace + 4 * (uint64_t)blk;
      rec[0] = t_begin; rec[1] = t_ready; rec[2] = wall_clock64();
      rec[3] = ((uint64_t)(uint32_t)pos << 32) | (uint32_t)blk;
    }
  }
}

extern "C" __global__ void __launch_bounds__(256, 4) opara_k_chain_f16_light(ChainArgs pa) { chain_body<true, true>(pa); }
extern "C" __global__ void __launch_bounds__(256, 2) opara_k_chain_f16_heavy(ChainArgs pa) { chain_body<true, false>(pa); }
extern "C" __global__ void __launch_bounds__(256, 4) opara_k_chain_f32_light(ChainArgs pa) { chain_body<false, true>(pa); }
extern "C" __global__ void __launch_bounds__(256, 2) opara_k_chain_f32_heavy(ChainArgs pa) { chain_body<false, false>(pa); }

// Dependency self-check: done-tokens per operator and a violation counter, in static
// device memory (nothing is allocated).
static __device__ int g_verify_tok[opara::kVerifyMaxOps];
static __device__ int g_verify_viol[4];   // violations, then 1 + operator and predecessor of the last one

extern "C" __global__ void opara_k_token(opara::TokenNodeArgs node) {
  const opara::TokenArgs &a = node.tok;
  if (threadIdx.x != 0) return;
  for (int i = 0; i < a.n_preds; ++i)
    if (__hip_atomic_load(&g_verify_tok[a.preds[i]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != a.epoch) {
      atomicAdd(&g_verify_viol[0], 1);
      g_verify_viol[1] = a.self + 1;
      g_verify_viol[2] = a.preds[i];
    }
  for (int i = 0; i < a.delay; ++i) __builtin_amdgcn_s_sleep(127);   // bounded: a few microseconds
  __hip_atomic_store(&g_verify_tok[a.self], a.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Workspace of the persistent executor for callers that cannot allocate device memory:
// counters, completion flags and operator records of up to kStaticWorkspaceMaxOps
// operators.  Every GPU the library runs on holds its own copy at its own address until
// the process ends; host code reaches it only through the address static_workspace()
// looks up (the array's name is a host-side stand-in, not a device address).
constexpr size_t kScratchBytes = 2560u * 1024u;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// Kernel without work: a pure dependency node (common root / common leaf of a capture).
extern "C" __global__ void opara_k_noop(int) {}

namespace opara {

// Operator-timeline buffer that launches and captures made from now on hand to their kernels.
static unsigned long long *g_host_op_trace = nullptr;

hipError_t launch_noop(hipStream_t s) {
  hipLaunchKernelGGL(opara_k_noop, dim3(1), dim3(64), 0, s, 0);
  return hipGetLastError();
}

namespace {
// What every planned kernel is given: its by-value record at offset 0, the launch's own arguments
// and the element-wise operator that follows; a kernel takes as many as it declares.
struct PlanParams {
  KernelArgs args;
  LaunchArgs launch;
  TailArgs tail;
  void *ptr[3];
  explicit PlanParams(const KernelPlan &p)
      : args(p.args), launch{p.tag, (int32_t)p.gx, (int32_t)p.gy, (int32_t)p.gz, g_host_op_trace}, tail(p.tail),
        ptr{&args, &launch, &tail} {}
  PlanParams(const PlanParams &) = delete;
};

// Size of a kernel's operator record.
size_t record_bytes(int id) {
  switch (id) {
#define X(name, A) case K_##name: return sizeof(A);
    OPARA_KERNEL_LIST(X)
#undef X
    default: return sizeof(KernelArgs);
  }
}

hipKernelNodeParams plan_node_params(const KernelPlan &p, PlanParams &params) {
  hipKernelNodeParams np = {};
  np.func = const_cast<void *>(kernel_symbol(p.kernel));
  np.gridDim = dim3(p.gx, p.gy, p.gz);
  np.blockDim = dim3(p.block);
  np.sharedMemBytes = 0;
  np.kernelParams = params.ptr;
  np.extra = nullptr;
  return np;
}
}  // namespace

hipError_t launch_plan(const KernelPlan &p, hipStream_t s) {
  PlanParams params(p);
  const void *func = kernel_symbol(p.kernel);
  if (!func) return hipErrorInvalidValue;
  return hipLaunchKernel(func, dim3(p.gx, p.gy, p.gz), dim3(p.block), params.ptr, 0, s);
}

hipError_t add_plan_node(hipGraph_t graph, const KernelPlan &p, const hipGraphNode_t *deps, size_t n_deps,
                         hipGraphNode_t *node) {
  PlanParams params(p);
  const hipKernelNodeParams np = plan_node_params(p, params);
  return np.func ? hipGraphAddKernelNode(node, graph, deps, n_deps, &np) : hipErrorInvalidValue;
}

hipError_t set_exec_node_plan(hipGraphExec_t exec, hipGraphNode_t node, const KernelPlan &p) {
  PlanParams params(p);
  const hipKernelNodeParams np = plan_node_params(p, params);
  return np.func ? hipGraphExecKernelNodeSetParams(exec, node, &np) : hipErrorInvalidValue;
}

hipError_t add_noop_node(hipGraph_t graph, const hipGraphNode_t *deps, size_t n_deps, hipGraphNode_t *node) {
  int zero = 0;
  void *kparams[1] = {&zero};
  hipKernelNodeParams np = {};
  np.func = (void *)opara_k_noop;
  np.gridDim = dim3(1);
  np.blockDim = dim3(64);
  np.kernelParams = kparams;
  return hipGraphAddKernelNode(node, graph, deps, n_deps, &np);
}

hipError_t add_token_node(hipGraph_t graph, const KernelPlan &p, const TokenArgs &t, const hipGraphNode_t *deps, size_t n_deps,
                          hipGraphNode_t *node) {
  const PlanParams params(p);
  const size_t record = record_bytes(p.kernel);
  TokenNodeArgs args = {};
  __builtin_memcpy(args.real, &params.args, record);
  __builtin_memcpy(args.real + record, &params.launch, sizeof(LaunchArgs));
  __builtin_memcpy(args.real + record + sizeof(LaunchArgs), &params.tail, sizeof(TailArgs));
  args.tok = t;
  void *kparams[1] = {&args};
  hipKernelNodeParams np = {};
  np.func = (void *)opara_k_token;
  np.gridDim = dim3(1);
  np.blockDim = dim3(64);
  np.kernelParams = kparams;
  return hipGraphAddKernelNode(node, graph, deps, n_deps, &np);
}

namespace {
void *group_func(bool f16, int flavor, bool traced) {
  static void *const f[2][2][3] = {
      {{(void *)opara_k_group_f32_stream, (void *)opara_k_group_f32_light, (void *)opara_k_group_f32_heavy},
       {(void *)opara_k_group_f16_stream, (void *)opara_k_group_f16_light, (void *)opara_k_group_f16_heavy}},
      {{(void *)opara_k_group_f32_stream_traced, (void *)opara_k_group_f32_light_traced, (void *)opara_k_group_f32_heavy_traced},
       {(void *)opara_k_group_f16_stream_traced, (void *)opara_k_group_f16_light_traced, (void *)opara_k_group_f16_heavy_traced}}};
  return f[traced ? 1 : 0][f16 ? 1 : 0][flavor < 0 ? 0 : flavor > 2 ? 2 : flavor];
}
}  // namespace

int group_flavor(int id) {
  switch (id) {
#define FCASE(name, Args, call) case K_##name:
    HEAVY_BODIES(FCASE, half_t, f16, 0) HEAVY_BODIES(FCASE, float, f32, 0) FAR_BODIES(FCASE, half_t, f16, 0) FAR_BODIES(FCASE, float, f32, 0) return 2;
    LIGHT_BODIES(FCASE, half_t, f16, 0) LIGHT_BODIES(FCASE, float, f32, 0) return 1;
#undef FCASE
    default: return id >= 0 && id < K_attention_f16 ? 0 : -1;     // merged operators run as launches of their own
  }
}

bool group_kernel_ok(int id, bool *light) {
  const int f = group_flavor(id);
  *light = f >= 0 && f < 2;
  return f >= 0;
}

// The limit is the kernel's, not the executor's: it is the same for every capture, so that none
// lowers it under an executor that is still in use.
hipError_t group_prepare() {
  for (int f16 = 0; f16 < 2; ++f16)
    for (int flavor = 0; flavor < 3; ++flavor)
      for (int traced = 0; traced < 2; ++traced) {
        hipError_t err = hipFuncSetAttribute(group_func(f16, flavor, traced), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLargestBody);
        if (err != hipSuccess) return err;
      }
  return hipSuccess;
}

hipError_t add_group_node(hipGraph_t graph, bool f16, int flavor, const GroupArgs &ga, uint32_t n_blocks,
                          uint32_t lds_bytes, const hipGraphNode_t *deps, size_t n_deps, hipGraphNode_t *node) {
  GroupArgs args = ga;
  void *kparams[1] = {&args};
  hipKernelNodeParams np = {};
  np.func = group_func(f16, flavor, ga.trace != nullptr);
  np.gridDim = dim3(n_blocks);
  np.blockDim = dim3(256);
  np.sharedMemBytes = lds_bytes;
  np.kernelParams = kparams;
  return hipGraphAddKernelNode(node, graph, deps, n_deps, &np);
}

hipError_t launch_group(bool f16, int flavor, const GroupArgs &ga, uint32_t n_blocks, uint32_t lds_bytes, hipStream_t s) {
  GroupArgs args = ga;
  void *kparams[1] = {&args};
  return hipLaunchKernel(group_func(f16, flavor, ga.trace != nullptr), dim3(n_blocks), dim3(256), kparams, lds_bytes, s);
}

namespace {
void *chain_func(bool f16, bool light) {
  return f16 ? (light ? (void *)opara_k_chain_f16_light : (void *)opara_k_chain_f16_heavy)
             : (light ? (void *)opara_k_chain_f32_light : (void *)opara_k_chain_f32_heavy);
}
}  // namespace

bool chain_kernel_ok(int id, bool *light) {
  return group_kernel_ok(id, light) && id != K_igemm_f16_far128x128 && id != K_igemm_f32_far128x128;
}

hipError_t chain_prepare() {
  for (int f16 = 0; f16 < 2; ++f16)
    for (int light = 0; light < 2; ++light) {
      hipError_t err = hipFuncSetAttribute(chain_func(f16, light), hipFuncAttributeMaxDynamicSharedMemorySize, kLdsLargestBody);
      if (err != hipSuccess) return err;
    }
  return hipSuccess;
}

hipError_t add_chain_node(hipGraph_t graph, bool f16, bool light, const ChainArgs &a, uint32_t lds_bytes,
                          const hipGraphNode_t *deps, size_t n_deps, hipGraphNode_t *node) {
  ChainArgs args = a;
  void *kparams[1] = {&args};
  hipKernelNodeParams np = {};
  np.func = chain_func(f16, light);
  np.gridDim = dim3((uint32_t)a.total);
  np.blockDim = dim3(256);
  np.sharedMemBytes = lds_bytes;
  np.kernelParams = kparams;
  return hipGraphAddKernelNode(node, graph, deps, n_deps, &np);
}

hipError_t launch_chain(bool f16, bool light, const ChainArgs &a, uint32_t lds_bytes, hipStream_t s) {
  const dim3 grid((uint32_t)a.total), block(256);
  if (f16) {
    if (light) hipLaunchKernelGGL(opara_k_chain_f16_light, grid, block, lds_bytes, s, a);
    else hipLaunchKernelGGL(opara_k_chain_f16_heavy, grid, block, lds_bytes, s, a);
  } else {
    if (light) hipLaunchKernelGGL(opara_k_chain_f32_light, grid, block, lds_bytes, s, a);
    else hipLaunchKernelGGL(opara_k_chain_f32_heavy, grid, block, lds_bytes, s, a);
  }
  return hipGetLastError();
}

int persist_kernel_id(int id) {
  switch (id) {
    case K_igemm_f16_t128x64: case K_igemm_f32_t128x64: case K_igemm_f16_t64x64: case K_igemm_f32_t64x64:
    case K_igemm_f16_t64x64_scalar: case K_igemm_f32_t64x64_scalar: case K_igemm_f16_direct4: case K_igemm_f32_direct4:
      return id;                          // one tile shape for every latency-oriented contraction
    default: return group_flavor(id) == 0 ? id : -1;
  }
}

bool kernel_is_f16(int id) {
  switch (id) {
#define X(name, A) case K_##name: return sizeof(#name) > 1 && __builtin_strstr(#name, "_f16") != nullptr;
    OPARA_KERNEL_LIST(X)
#undef X
    default: return false;
  }
}

namespace {
typedef void (*PersistKernel)(PersistArgs);
PersistKernel persist_func(bool f16, bool tiled) {
  return f16 ? (tiled ? opara_k_persist_f16_tiled : opara_k_persist_f16) : (tiled ? opara_k_persist_f32_tiled : opara_k_persist_f32);
}
}  // namespace

hipError_t persist_max_workgroups(bool f16, bool tiled, uint32_t lds_bytes, uint32_t *n_workgroups) {
  int dev = 0, cus = 0, per_cu = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  err = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (err != hipSuccess) return err;
  err = hipFuncSetAttribute((const void *)persist_func(f16, tiled), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)kPersistMaxLds);   // for every executor alike
  if (err != hipSuccess) return err;
  err = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persist_func(f16, tiled), 256, lds_bytes);
  if (err != hipSuccess) return err;
  *n_workgroups = (uint32_t)(per_cu > 0 ? per_cu : 0) * (uint32_t)cus;
  return hipSuccess;
}

hipError_t add_persist_node(hipGraph_t graph, bool f16, bool tiled, const PersistArgs &a, uint32_t n_workgroups,
                            uint32_t lds_bytes, const hipGraphNode_t *deps, size_t n_deps, hipGraphNode_t *node) {
  PersistArgs args = a;
  void *kparams[1] = {&args};
  hipKernelNodeParams np = {};
  np.func = (void *)persist_func(f16, tiled);
  np.gridDim = dim3(n_workgroups);
  np.blockDim = dim3(256);
  np.sharedMemBytes = lds_bytes;
  np.kernelParams = kparams;
  return hipGraphAddKernelNode(node, graph, deps, n_deps, &np);
}

hipError_t launch_persist(bool f16, bool tiled, const PersistArgs &a, uint32_t n_workgroups, uint32_t lds_bytes, hipStream_t s) {
  hipLaunchKernelGGL(persist_func(f16, tiled), dim3(n_workgroups), dim3(256), lds_bytes, s, a);
  return hipGetLastError();
}

hipError_t static_workspace(void **ptr, size_t *bytes) {
  constexpr int kMaxDevices = 64;
  static void *addr[kMaxDevices];          // per device, written once (the lookup is idempotent)
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  void *p = __atomic_load_n(&addr[dev], __ATOMIC_ACQUIRE);
  if (!p) {
    err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (err != hipSuccess) return err;
    if (!p) return hipErrorInvalidSymbol;
    __atomic_store_n(&addr[dev], p, __ATOMIC_RELEASE);
  }
  *ptr = p;
  *bytes = kScratchBytes;
  return hipSuccess;
}

hipError_t set_op_trace(void *device_buffer) {
  g_host_op_trace = (unsigned long long *)device_buffer;
  return hipSuccess;
}

void *current_op_trace() { return g_host_op_trace; }

hipError_t verify_reset(hipStream_t s) {
  void *tok = nullptr, *viol = nullptr;
  hipError_t err = hipGetSymbolAddress(&tok, HIP_SYMBOL(g_verify_tok));
  if (err != hipSuccess) return err;
  err = hipGetSymbolAddress(&viol, HIP_SYMBOL(g_verify_viol));
  if (err != hipSuccess) return err;
  err = hipMemsetAsync(tok, 0, sizeof(int) * kVerifyMaxOps, s);
  if (err != hipSuccess) return err;
  return hipMemsetAsync(viol, 0, sizeof(int) * 4, s);
}

hipError_t verify_read(hipStream_t s, int *viol, int *op, int *pred) {
  void *p = nullptr;
  int v[4] = {0, 0, 0, 0};
  hipError_t err = hipGetSymbolAddress(&p, HIP_SYMBOL(g_verify_viol));
  if (err != hipSuccess) return err;
  err = hipMemcpyAsync(v, p, sizeof v, hipMemcpyDeviceToHost, s);
  if (err != hipSuccess) return err;
  err = hipStreamSynchronize(s);
  *viol = v[0];
  if (op) *op = v[1] - 1;
  if (pred) *pred = v[2];
  return err;
}

const void *kernel_symbol(int id) {
  switch (id) {
#define X(name, A) \
  case K_##name:   \
    return (const void *)opara_k_##name;
    OPARA_KERNEL_LIST(X)
#undef X
    default:
      return nullptr;
  }
}

}  // namespace opara
