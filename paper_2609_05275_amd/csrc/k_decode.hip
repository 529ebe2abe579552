// Kernels of incremental (KV-cached) decoding: a few new rows per sequence
// go through a layer whose keys and values of earlier positions are cached.
// Both hot kernels are bound by HBM reads: the fused projection (below) reads
// each weight matrix once, the decode attention each cached key/value row.
//
// Skinny GEMM (the standalone entry point; M <= 64 rows, bf16, v_mfma_f32_32x32x16_bf16): one wave owns
// 32 output columns; the four waves of a workgroup (and, with ksplit > 1,
// several workgroups) take interleaved 64-wide k chunks of the same columns.
// Within a chunk the k index of the four MFMAs is permuted so that each lane
// reads 64 contiguous bytes of its row: lane half h, MFMA s holds
// k = 64c + 32h + 8s + e (e < 8), in A and W alike, which leaves the
// contraction unchanged.  The waves' accumulators are summed in LDS in wave
// order; split workgroups write float32 partials summed in split order by a
// second kernel, so results do not depend on timing.  (A last-arriving
// workgroup doing that sum needs device-scope fences, which on this chip
// write back and invalidate the per-XCD L2 and cost far more than the
// second launch.)
//
// Decode attention: one workgroup per (chunk of keys, head, sequence), scores
// in base 2 with the causal cut (key <= query position) and the ALiBi bias.  A
// combine kernel merges the chunks with the usual max/sum rescaling and writes
// bf16; a single chunk writes its result itself.
#include "ld_internal.h"

namespace ld {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kSkWaves = 4;
constexpr int kSkChunk = 64;

__device__ __forceinline__ bf16x8 zero8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = static_cast<bf16>(0.f);
  return z;
}

__device__ __forceinline__ bf16x8 load8(const bf16* p) { return *reinterpret_cast<const bf16x8*>(p); }

__device__ __forceinline__ void skinny_store(const SkinnyArgs& g, int m, int n, float sum) {
  float v = g.alpha * sum;
  if (g.R) v += static_cast<float>(static_cast<const bf16*>(g.R)[static_cast<int64_t>(m) * g.ldr + n]);
  const bf16 o = static_cast<bf16>(v);
  static_cast<bf16*>(g.C)[static_cast<int64_t>(m) * g.ldc + n] = o;
  if (g.kv && n >= g.kv_d) {
    const int64_t b = m / g.kv_n, j = m % g.kv_n;
    static_cast<bf16*>(g.kv)[(b * g.kv_s_max + g.kv_pos + j) * 2 * g.kv_d + (n - g.kv_d)] = o;
  }
}

template <int MB>
__global__ __launch_bounds__(256) void ld_gemm_bf16_skinny(SkinnyArgs g) {
  __shared__ float red[kSkWaves * MB * 16 * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 31, h = lane >> 5;
  const int n0 = blockIdx.x * 32;
  const int nchunks = (g.K + kSkChunk - 1) / kSkChunk;
  const int workers = kSkWaves * gridDim.y;
  const bf16* A = static_cast<const bf16*>(g.A);
  const bf16* W = static_cast<const bf16*>(g.W);
  const bool nvalid = n0 + li < g.N;
  const bf16* wrow = W + static_cast<int64_t>(nvalid ? n0 + li : 0) * g.ldw + 32 * h;
  const bf16* arow[MB];
  bool mvalid[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    mvalid[mb] = mb * 32 + li < g.M;
    arow[mb] = A + static_cast<int64_t>(mvalid[mb] ? mb * 32 + li : 0) * g.lda + 32 * h;
  }
  floatx16 acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[mb][v] = 0.f;

  // U chunks per pass, all loaded before their MFMAs (chunks past the end
  // load zeros, so the MFMAs need no branch)
  constexpr int U = MB == 1 ? 4 : 2;
  for (int c0 = blockIdx.y * kSkWaves + wave; c0 < nchunks; c0 += U * workers) {
    bf16x8 b[U][4], a[U][MB][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kc = (c0 + u * workers) * kSkChunk;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const bool kv = kc + 32 * h + 8 * s < g.K;   // K % 8 == 0: the whole 8 are in range
        b[u][s] = (nvalid && kv) ? load8(wrow + kc + 8 * s) : zero8();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          a[u][mb][s] = (mvalid[mb] && kv) ? load8(arow[mb] + kc + 8 * s) : zero8();
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          acc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[u][mb][s], b[u][s], acc[mb], 0, 0, 0);
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) red[((wave * MB + mb) * 16 + v) * 64 + lane] = acc[mb][v];
  __syncthreads();
  constexpr int kElems = MB * 16 * 64;
  for (int e = threadIdx.x; e < kElems; e += 256) {
    float sum = red[e];
#pragma unroll
    for (int w = 1; w < kSkWaves; ++w) sum += red[w * kElems + e];
    const int l = e & 63, v = (e >> 6) & 15, mb = e >> 10;
    const int m = mb * 32 + 8 * (v >> 2) + 4 * (l >> 5) + (v & 3);
    const int n = n0 + (l & 31);
    if (m < g.M && n < g.N) {
      if (gridDim.y > 1 || g.part_only)
        g.part[(static_cast<int64_t>(blockIdx.y) * g.M + m) * g.N + n] = sum;
      else
        skinny_store(g, m, n, sum);
    }
  }
}

__global__ __launch_bounds__(256) void ld_skinny_reduce_k(SkinnyArgs g, int ksplit) {
  const int64_t total = static_cast<int64_t>(g.M) * g.N;
  for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < total; i += gridDim.x * 256ll) {
    float sum = g.part[i];
    for (int s = 1; s < ksplit; ++s) sum += g.part[s * total + i];
    skinny_store(g, static_cast<int>(i / g.N), static_cast<int>(i % g.N), sum);
  }
}

__device__ __forceinline__ float bf16r(float x) { return static_cast<float>(static_cast<bf16>(x)); }

// Split-K sums (split order) of one row of a skinny GEMM with alpha and the
// residual, stored as C, then (when a gain is given) the RMSNorm of the
// stored row (sum of squares over the workgroup in a fixed order):
// h = bf16(C rstd gain).  One workgroup of 1024 threads per row.
__global__ __launch_bounds__(1024) void ld_skinny_reduce_norm_k(SkinnyArgs g, int ksplit, const bf16* gain,
                                                                 float eps, bf16* h) {
  constexpr int kPer = 4;  // columns per thread and pass: one pass up to 4096 columns
  __shared__ float wsum[16];
  const int m = blockIdx.x, tid = threadIdx.x;
  const int64_t mn = static_cast<int64_t>(g.M) * g.N;
  const float* prow = g.part + static_cast<int64_t>(m) * g.N;
  bf16* C = static_cast<bf16*>(g.C) + static_cast<int64_t>(m) * g.ldc;
  const bf16* R = g.R ? static_cast<const bf16*>(g.R) + static_cast<int64_t>(m) * g.ldr : nullptr;
  float ss = 0.f;
  for (int n0 = 0; n0 < g.N; n0 += 1024 * kPer) {
    float sum[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) sum[i] = 0.f;
    // the splits in order; every column's loads of a split are independent
#pragma unroll 2
    for (int sp = 0; sp < ksplit; ++sp)
#pragma unroll
      for (int i = 0; i < kPer; ++i) {
        const int n = n0 + i * 1024 + tid;
        if (n < g.N) sum[i] += prow[sp * mn + n];
      }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int n = n0 + i * 1024 + tid;
      if (n < g.N) {
        const bf16 o = static_cast<bf16>(g.alpha * sum[i] + (R ? static_cast<float>(R[n]) : 0.f));
        C[n] = o;
        const float of = static_cast<float>(o);
        ss = __builtin_fmaf(of, of, ss);
      }
    }
  }
  if (!gain) return;  // no norm follows (workgroup-uniform)
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, 64);
  if ((tid & 63) == 0) wsum[tid >> 6] = ss;
  __syncthreads();
  float tot = 0.f;
#pragma unroll
  for (int w = 0; w < 16; ++w) tot += wsum[w];
  const float rstd = rsqrtf(tot / static_cast<float>(g.N) + eps);
  bf16* hr = h + static_cast<int64_t>(m) * g.N;
  for (int n = tid; n < g.N; n += 1024)  // this thread's own stores, read back
    hr[n] = static_cast<bf16>(static_cast<float>(C[n]) * rstd * static_cast<float>(gain[n]));
}

// The FFN activation from a skinny GEMM's partials: u (and v = column f + n
// for SwiGLU) rounded to bf16 as stored outputs would be, s = act(u, v).
__global__ __launch_bounds__(256) void ld_skinny_reduce_act_k(SkinnyArgs g, int ksplit, int act, int f, bf16* so) {
  const int64_t mn = static_cast<int64_t>(g.M) * g.N, total = static_cast<int64_t>(g.M) * f;
  for (int64_t i = blockIdx.x * 256ll + threadIdx.x; i < total; i += gridDim.x * 256ll) {
    const int64_t m = i / f, n = i % f, iu = m * g.N + n;
    float su = g.part[iu];
#pragma unroll 4
    for (int sp = 1; sp < ksplit; ++sp) su += g.part[sp * mn + iu];
    const float u = bf16r(g.alpha * su);
    float out;
    if (act == kDecActSwiglu) {
      float sv = g.part[iu + f];
#pragma unroll 4
      for (int sp = 1; sp < ksplit; ++sp) sv += g.part[sp * mn + iu + f];
      out = swiglu_fwd_f(u, bf16r(g.alpha * sv));
    } else {
      const float z = fmaxf(u, 0.f);
      out = z * z;
    }
    so[m * f + n] = static_cast<bf16>(out);
  }
}

// ------------------------------------------------ fused decode projection
// At most 48 rows.  Bound by the weight stream: W is read once, and the
// rest is kept out of its way.  A tile is 8 output columns (8 rows of W; with
// SwiGLU the 8 gate rows and the 8 up rows of those columns) over the whole
// k range, so every column is finished in one workgroup (no split-K partials,
// no reduction launch) and N = 2048 still spreads over 256 workgroups.
//
// Lane l reads 16 bytes of row l % 8 at k = 64c + 32 ((l / 8) % 2) + 8 (l / 16),
// of W and of the activations alike, so a load instruction takes 8 whole
// 128-byte lines.  As operands of v_mfma_f32_16x16x32_bf16 the lanes hold 8
// rows of W (A) and 8 rows of activations (B), each twice: rows 0-7 with the
// first 32 k of the chunk, rows 8-15 with the last 32.  One product then gives
// both halves on its diagonal 8x8 blocks, which are added; the off-diagonal
// blocks mix the halves and are dropped.  (Dot products on the vector ALU,
// which this replaces, read every row of A from LDS once per 8 columns: at 8
// rows the LDS, at one row the padding to 8 rows, cost more than the weights.
// 1B shape at 8 rows: QKV 14.8 -> 8.4 us, gate/up 18.5 -> 10.9, output 6.6 -> 5.0,
// down 11.6 -> 10.4, for 25, 45, 8 and 23 MB of weights.  At 48 rows, against
// split-K GEMMs and their reductions: the four projections with their norms and
// activation 95 -> 68 us; there every CU reading all the activations is what
// bounds it, at about 15 bytes a clock.)
//
// The waves take interleaved chunks.  ld_gemm_bf16_dec keeps its waves'
// activations in registers (K <= 2048 at up to 48 rows, 4096 at up to 16):
// loaded straight from memory in operand layout and used for every tile the workgroup takes in turn, so a CU reads A once; the
// first two tiles' weights are requested before anything waits where the
// registers allow.  With a gain, RMSNorm costs the operand one multiplication:
// the sums of squares are the diagonals of x x^T on the matrix cores, exchanged
// with the first tile's sums, and 1/rms scales the outputs.  (Squares and both
// scalings on the vector ALU, and a barrier before the first product: QKV and
// gate/up 19.0 and 25.1 us at 48 rows, now 16.8 and 21.1; 9.4 and 12.0 at 8, now
// 8.4 and 10.9.)  ld_gemm_bf16_dec_long streams the activations beside the
// weights.
//
// Partial sums go over the waves in wave order through LDS; the epilogue
// applies alpha and the residual (and copies key/value columns to the cache)
// or the activation, rounding u and v to bf16 first as stored outputs would be.

constexpr int kDecCols = 8;   // output columns per tile
constexpr int kDecCus = 256;  // compute units

typedef int int4v __attribute__((ext_vector_type(4)));

// Sums of the waves' products of one tile: red[wave][j][m][8 columns], MB
// blocks of 8 rows.
template <int MB, int NR>
constexpr int dec_red_floats() { return NR * MB * 8 * kDecCols; }

// Lane l of a product holds D rows 4 (l / 16) + e of column l % 16: the first
// 32 k's block in the lanes with bits 3 and 5 clear, the last 32 k's in those
// with both set.  Their sum goes to the wave's block of `red`.
template <int MB, int NR>
__device__ __forceinline__ void dec_put(float* red, const floatx4 (&acc)[NR][MB], int lane) {
#pragma unroll
  for (int j = 0; j < NR; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      floatx4 v = acc[j][mb];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += __shfl_xor(v[e], 40, 64);
      if ((lane & 40) == 0)
        *reinterpret_cast<floatx4*>(red + ((j * MB + mb) * 8 + (lane & 7)) * kDecCols + 4 * (lane >> 4)) = v;
    }
}

// Element (row em, column en) of the output from the waves' sums.
template <int MB, int ACT, int NW>
__device__ __forceinline__ void dec_finish(const SkinnyArgs& g, const float* red, int em, int c, int en, uint16_t resid,
                                           float alpha) {
  constexpr int NR = ACT == kDecActSwiglu ? 2 : 1;
  constexpr int kWave = dec_red_floats<MB, NR>();
  const int at = em * kDecCols + c;
  float s0 = red[at], s1 = 0.f;
#pragma unroll
  for (int w = 1; w < NW; ++w) s0 += red[w * kWave + at];
  if constexpr (NR == 2) {
    s1 = red[kWave / 2 + at];
#pragma unroll
    for (int w = 1; w < NW; ++w) s1 += red[w * kWave + kWave / 2 + at];
  }
  bf16* C = static_cast<bf16*>(g.C) + static_cast<int64_t>(em) * g.ldc + en;
  if constexpr (ACT == kDecActSwiglu) {
    *C = static_cast<bf16>(swiglu_fwd_f(bf16r(alpha * s0), bf16r(alpha * s1)));
  } else if constexpr (ACT == kDecActRelu2) {
    const float z = fmaxf(bf16r(alpha * s0), 0.f);
    *C = static_cast<bf16>(z * z);
  } else {
    const bf16 o = static_cast<bf16>(alpha * s0 + (g.R ? static_cast<float>(__builtin_bit_cast(bf16, resid)) : 0.f));
    *C = o;
    if (g.kv && en >= g.kv_d) {
      const int64_t b = em / g.kv_n, jj = em % g.kv_n;
      static_cast<bf16*>(g.kv)[(b * g.kv_s_max + g.kv_pos + jj) * 2 * g.kv_d + (en - g.kv_d)] = o;
    }
  }
}

// The residual of an output element as stored, converted where it is used
// and loaded without a branch, so that nothing waits for it (and for the loads
// before it) earlier.  Without a residual: any readable element.
__device__ __forceinline__ uint16_t dec_resid(const SkinnyArgs& g, int em, int en) {
  const uint16_t* p = static_cast<const uint16_t*>(g.R ? g.R : g.A);
  return p[g.R ? static_cast<int64_t>(min(em, g.M - 1)) * g.ldr + min(en, g.N - 1) : 0];
}

// Zeroes what was loaded from a clamped address: the lane's 8 values at k >= K.
__device__ __forceinline__ void dec_mask(bf16x8& v, bool keep) {
  int4v t = __builtin_bit_cast(int4v, v);
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = keep ? t[i] : 0;
  v = __builtin_bit_cast(bf16x8, t);
}

// The wave's number.  It decides which chunks a wave takes, so neighbouring
// workgroups of an XCD (every 8th) count from different waves: started in step,
// all would ask the same few L2 channels for the same lines of A first.  Sums
// go by this number, so the results do not depend on it.  QKV and gate/up of
// the 1B shape: 8.1 -> 7.5 and 11.8 -> 11.1 us at one row, 9.1 -> 8.4 and 11.7 ->
// 10.8 us at 8.
template <int NW>
__device__ __forceinline__ int dec_wave() {
  return __builtin_amdgcn_readfirstlane((threadIdx.x >> 6) + (blockIdx.x >> 3)) & (NW - 1);
}

// K <= 64 NW CPW; MB blocks of 8 rows; one thread per output element of a tile
// (NW * 64 >= 64 MB).
template <int MB, int ACT, bool NORM, int NW, int CPW>
__global__ __launch_bounds__(NW * 64) void ld_gemm_bf16_dec(SkinnyArgs g) {
  constexpr int NR = ACT == kDecActSwiglu ? 2 : 1;  // W rows per lane
  constexpr int kRed = NW * dec_red_floats<MB, NR>();
  static_assert(NW * 64 >= MB * 8 * kDecCols, "a thread per output element");
  __shared__ __align__(16) float red[2][kRed];
  __shared__ float ssq[NORM ? NW : 1][MB * 8];
  // the second tile's weights go out before the normalisation if the registers allow
  constexpr bool kTwo = CPW * NR <= 8;  // two tiles' weights in hand, else one
  constexpr bool kBoth = kTwo && (!NORM || MB <= 2 || NR == 1);
  const int M = g.M, N = g.N, K = g.K;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = dec_wave<NW>();
  const int tiles = (N + kDecCols - 1) / kDecCols;
  const int lk = 32 * ((lane >> 3) & 1) + 8 * (lane >> 4);  // the lane's k of a chunk
  const bf16* W = static_cast<const bf16*>(g.W);

  typedef bf16x8 WBuf[CPW][NR];
  auto load_w = [&](WBuf& wb, int tile) {
    // no branch around a load (the compiler would wait at each): columns past
    // N repeat the last, k past K the row's start
    const int col = min(tile * kDecCols + (lane & 7), N - 1);
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const bf16* wrow = W + static_cast<int64_t>(col + j * N) * g.ldw;
#pragma unroll
      for (int u = 0; u < CPW; ++u) {
        const int k = (wave + NW * u) * 64 + lk;
        wb[u][j] = load8(wrow + (k < K ? k : 0));
      }
    }
  };
  WBuf w0, w1;
  load_w(w0, blockIdx.x);
  if (kBoth) load_w(w1, blockIdx.x + gridDim.x);
  const int em = tid / kDecCols, c = tid % kDecCols;  // the thread's output element of a tile
  const bool erow = em < M;
  uint16_t r0 = 0, r1 = 0;  // its residual, of the two tiles in hand
  if (ACT == kDecActNone) {
    r0 = dec_resid(g, em, blockIdx.x * kDecCols + c);
    r1 = dec_resid(g, em, (blockIdx.x + gridDim.x) * kDecCols + c);
  }

  // this wave's gains and activations in operand layout (rows past M repeat the last)
  bf16x8 gv[CPW], x[CPW][MB];
  if constexpr (NORM) {
#pragma unroll
    for (int u = 0; u < CPW; ++u) {
      const int k = (wave + NW * u) * 64 + lk;
      gv[u] = load8(static_cast<const bf16*>(g.g) + (k < K ? k : 0));
    }
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const bf16* xr = static_cast<const bf16*>(g.A) + static_cast<int64_t>(min(mb * 8 + (lane & 7), M - 1)) * g.lda;
#pragma unroll
    for (int u = 0; u < CPW; ++u) {
      const int k = (wave + NW * u) * 64 + lk;
      x[u][mb] = load8(xr + (k < K ? k : 0));
    }
  }
#pragma unroll
  for (int u = 0; u < CPW; ++u)
    if ((wave + NW * u) * 64 + 64 > K) {  // wave-uniform
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) dec_mask(x[u][mb], (wave + NW * u) * 64 + lk < K);
    }
  if constexpr (NORM) {
    // Sums of squares from the products of the rows with themselves (the
    // diagonals of the two blocks); the gain goes on the operand, 1/rms on the
    // outputs, so nothing here waits for the other waves.
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      floatx4 q{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < CPW; ++u) q = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u][mb], x[u][mb], q, 0, 0, 0);
      // lane l: D rows 4 (l / 16) + e of column l % 16
      const int e = lane & 3;
      float ss = e == 0 ? q[0] : e == 1 ? q[1] : e == 2 ? q[2] : q[3];
      ss += __shfl_xor(ss, 40, 64);
      if ((lane & 40) == 0 && (lane & 15) >> 2 == lane >> 4) ssq[wave][mb * 8 + (lane & 7)] = ss;
    }
#pragma unroll
    for (int u = 0; u < CPW; ++u) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 8; ++i)
          x[u][mb][i] = static_cast<bf16>(static_cast<float>(x[u][mb][i]) * static_cast<float>(gv[u][i]));
      if ((wave + NW * u) * 64 + 64 > K) {  // wave-uniform
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) dec_mask(x[u][mb], (wave + NW * u) * 64 + lk < K);
      }
    }
  }
  if (kTwo && !kBoth) load_w(w1, blockIdx.x + gridDim.x);

  // one tile: products, the request of the buffer's next tile, the waves' sums
  // into red[buf], and after the barrier the outputs (the other buffer's
  // readers are past the barrier before it is written again)
  float scale = g.alpha;
  auto do_tile = [&](WBuf& wb, int tile, int next, int buf, uint16_t& resid) {
    floatx4 acc[NR][MB];
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[j][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < CPW; ++u) {
      if ((wave + NW * u) * 64 + 64 > K) {  // wave-uniform: x is zero there, and W must not be inf or NaN
#pragma unroll
        for (int j = 0; j < NR; ++j) dec_mask(wb[u][j], (wave + NW * u) * 64 + lk < K);
      }
#pragma unroll
      for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          acc[j][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[u][j], x[u][mb], acc[j][mb], 0, 0, 0);
    }
    const uint16_t r = resid;
    if (next < tiles) {
      load_w(wb, next);
      if (ACT == kDecActNone) resid = dec_resid(g, em, next * kDecCols + c);
    }
    dec_put<MB, NR>(red[buf] + wave * dec_red_floats<MB, NR>(), acc, lane);
    __syncthreads();
    const int en = tile * kDecCols + c;
    if (erow && en < N) {
      if (NORM && tile == static_cast<int>(blockIdx.x)) {
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) tot += ssq[w][em];
        scale = g.alpha * rsqrtf(tot / static_cast<float>(K) + g.eps);
      }
      dec_finish<MB, ACT, NW>(g, red[buf], em, c, en, r, scale);
    }
  };
  const int step = gridDim.x;
  if constexpr (kTwo) {
    for (int tile = blockIdx.x; tile < tiles; tile += 2 * step) {
      do_tile(w0, tile, tile + 2 * step, 0, r0);
      if (tile + step < tiles) do_tile(w1, tile + step, tile + 3 * step, 1, r1);
    }
  } else {
    int buf = 0;
    for (int tile = blockIdx.x; tile < tiles; tile += step, buf ^= 1) do_tile(w0, tile, tile + step, buf, r0);
  }
}

// Any K: weights and activations streamed in passes of U chunks per wave, the
// next pass's loads in flight while one is used.  One tile per workgroup.
template <int MB, int ACT, int NW, int U>
__global__ __launch_bounds__(NW * 64) void ld_gemm_bf16_dec_long(SkinnyArgs g) {
  constexpr int NR = ACT == kDecActSwiglu ? 2 : 1;
  static_assert(NW * 64 >= MB * 8 * kDecCols, "a thread per output element");
  __shared__ __align__(16) float red[NW * dec_red_floats<MB, NR>()];
  const int M = g.M, N = g.N, K = g.K;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = dec_wave<NW>();
  const int lk = 32 * ((lane >> 3) & 1) + 8 * (lane >> 4);
  const int col = min(blockIdx.x * kDecCols + (lane & 7), N - 1);  // columns past N repeat the last
  const bf16 *wrow[NR], *xrow[MB];
#pragma unroll
  for (int j = 0; j < NR; ++j) wrow[j] = static_cast<const bf16*>(g.W) + static_cast<int64_t>(col + j * N) * g.ldw;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
    xrow[mb] = static_cast<const bf16*>(g.A) + static_cast<int64_t>(min(mb * 8 + (lane & 7), M - 1)) * g.lda;
  struct Pass {
    bf16x8 w[U][NR], x[U][MB];
  };
  // Chunks c0, c0 + NW, ...; k past K reads the row's start (no branch around
  // a load, where the compiler would wait), and `use` drops it.
  auto load = [&](Pass& p, int c0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kc = (c0 + NW * u) * 64, k = kc + lk < K ? kc + lk : 0;
#pragma unroll
      for (int j = 0; j < NR; ++j) p.w[u][j] = load8(wrow[j] + k);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) p.x[u][mb] = load8(xrow[mb] + k);
    }
  };
  floatx4 acc[NR][MB];
#pragma unroll
  for (int j = 0; j < NR; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[j][mb] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto use = [&](Pass& p, int c0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kc = (c0 + NW * u) * 64;
      if (kc + 64 > K) {  // wave-uniform
#pragma unroll
        for (int j = 0; j < NR; ++j) dec_mask(p.w[u][j], kc + lk < K);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) dec_mask(p.x[u][mb], kc + lk < K);
      }
#pragma unroll
      for (int j = 0; j < NR; ++j)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
          acc[j][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p.w[u][j], p.x[u][mb], acc[j][mb], 0, 0, 0);
    }
  };
  const int nchunks = (K + 63) >> 6;
  Pass p0, p1;
  load(p0, wave);
  load(p1, wave + U * NW);
  const int em = tid / kDecCols, c = tid % kDecCols, en = blockIdx.x * kDecCols + c;
  const bool eval = em < M && en < N;
  uint16_t resid = 0;
  if (ACT == kDecActNone) resid = dec_resid(g, em, en);
  for (int c0 = wave; c0 < nchunks; c0 += 2 * U * NW) {
    use(p0, c0);
    if (c0 + 2 * U * NW < nchunks) load(p0, c0 + 2 * U * NW);
    use(p1, c0 + U * NW);
    if (c0 + 3 * U * NW < nchunks) load(p1, c0 + 3 * U * NW);
  }
  dec_put<MB, NR>(red + wave * dec_red_floats<MB, NR>(), acc, lane);
  __syncthreads();
  if (eval) dec_finish<MB, ACT, NW>(g, red, em, c, en, resid, g.alpha);
}

// ------------------------------------------------------------ KV store

__global__ __launch_bounds__(256) void ld_kv_store_k(KvArgs a) {
  const int64_t per_row = (2ll * a.d) / 8;
  const int64_t total = static_cast<int64_t>(a.n_seq) * a.n * per_row;
  const bf16* src = static_cast<const bf16*>(a.qkv);
  bf16* dst = static_cast<bf16*>(a.cache);
  for (int64_t id = blockIdx.x * 256ll + threadIdx.x; id < total; id += gridDim.x * 256ll) {
    const int64_t r = id / per_row, c = (id % per_row) * 8;
    const int64_t b = r / a.n, j = r % a.n;
    const bf16x8 v = load8(src + r * a.ld_qkv + a.d + c);
    *reinterpret_cast<bf16x8*>(dst + ((b * a.s_max + a.pos + j) * 2 * a.d) + c) = v;
  }
}

// ------------------------------------------------------ decode attention

// A workgroup takes a chunk of 64 KB keys of one head and sequence, each of
// its eight waves 8 KB of them from load to weighted sum on its own; the
// waves meet once, to add up.  Bound by the cache stream: all loads of a
// wave, keys and values, go out before anything waits, so what it holds in
// registers is what it has in flight (32 keys at most: two workgroups fit a
// CU).
//
// Scores S^T = K Q^T on the matrix cores (16x16x32), 8 keys a time.  Lane l
// loads 16 bytes of key l % 8 at dimension 64 s + 32 ((l / 8) % 2) + 8 (l / 16),
// so an instruction takes 8 whole 128-byte lines (the load cost goes by the
// lines touched).  As A operand its lanes hold the keys twice, rows 0-7 with
// dimensions 0-31 of the 64 and rows 8-15 with 32-63, so each load feeds two
// products, against the query rows' (B operand, row l % 16, rows past n_new
// repeating the last) first and last 32 dimensions.  Of a product's 4 keys per
// lane, lanes l and l ^ 32 add up two each: lane group g = l / 16 ends with
// keys 4 (g % 2) + 2 (g / 2) + t, t < 2, of the 8.
//
// The values are loaded to match: group g's lanes hold those keys' rows, DH/16
// dimensions each.  Several query rows: P is then the A operand and V the B
// operand of v_mfma_f32_16x16x4_f32 (float32 in, nothing rounded) as they
// stand, column n of product e being dimension n DH/16 + e.  One query row:
// every lane has its key's probability, and multiplies it in itself.
//
// The split of the cache into chunks is dec_attn_blocks's.  Measured per layer
// of 16 heads of 128, before -> now: one row over 778 keys 9.2 -> 4.3 us; six
// rows of 8 sequences over 1506 keys 34.2 -> 23.3 us (4.2 TB/s of cache); one
// row of 8 sequences over 2048 keys 27.4 -> 25.9 us (5.2 TB/s), its combine 5.5 ->
// 4.8.  Before, waves of
// 64 keys loaded the values after the scores, the probabilities went through
// LDS, and the sum over keys through lane exchanges.
template <int DH, int NQ, int KB>
__global__ __launch_bounds__(512) void ld_attn_decode_bf16(DecAttnArgs a) {
  constexpr int EPL = DH / 16;  // dimensions per lane of a value row
  typedef __bf16 VRow __attribute__((ext_vector_type(EPL)));
  __shared__ float ml[8][NQ][2];
  __shared__ __align__(16) float red[8][NQ][DH];
  const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int64_t d = static_cast<int64_t>(a.H) * DH, row2 = 2 * d;
  const int nk = a.pos + a.n_new;
  const int k0 = (c * 8 + wave) * 8 * KB;
  const int kv0 = k0 + 4 * (g & 1) + 2 * (g >> 1);  // the lane's keys: kv0 + 8 kb + t
  const float al2 = a.alibi ? alibi_slope(h, a.H) * kLog2e : 0.f, sl2 = a.scale * kLog2e;
  const bf16* q = static_cast<const bf16*>(a.qkv) + h * DH +
                  (static_cast<int64_t>(b) * a.n_new + min(n, a.n_new - 1)) * a.ld_qkv;
  const bf16* cache = static_cast<const bf16*>(a.cache) + static_cast<int64_t>(b) * a.s_max * row2 + h * DH;

  // keys past the last position read row 0
  bf16x8 qf[DH / 64][2], kf[KB][DH / 64];
  VRow vr[KB][2];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int kk = k0 + kb * 8 + (lane & 7);
    const bf16* kp = cache + static_cast<int64_t>(kk < nk ? kk : 0) * row2 + 32 * ((lane >> 3) & 1) + 8 * g;
#pragma unroll
    for (int s = 0; s < DH / 64; ++s) kf[kb][s] = load8(kp + 64 * s);
  }
#pragma unroll
  for (int s = 0; s < DH / 64; ++s)
#pragma unroll
    for (int e = 0; e < 2; ++e) qf[s][e] = load8(q + 64 * s + 32 * e + 8 * g);
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kk = kv0 + 8 * kb + t;
      vr[kb][t] = *reinterpret_cast<const VRow*>(cache + static_cast<int64_t>(kk < nk ? kk : 0) * row2 + d + EPL * n);
    }
  __builtin_amdgcn_sched_barrier(0);  // the value loads stay ahead of the scores
  if (k0 + 8 * KB > nk) {  // wave-uniform: what was read in place of keys past the last counts as zeros
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (kv0 + 8 * kb + t >= nk) vr[kb][t] = static_cast<bf16>(0.f);
  }

  const int qpos = a.pos + (NQ == 1 ? 0 : n);
  float p[KB][2];
  float m = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    floatx4 s0{0.f, 0.f, 0.f, 0.f}, s1{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < DH / 64; ++s) {
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][s], qf[s][0], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[kb][s], qf[s][1], s1, 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {  // groups 0, 1: rows 0-7 of s0; 2, 3: rows 8-15 of s1
      const float give = g < 2 ? s0[2 + t] : s1[t], keep = g < 2 ? s0[t] : s1[2 + t];
      const float x = keep + __shfl_xor(give, 32, 64);
      const int kk = kv0 + 8 * kb + t;
      p[kb][t] = (kk < nk && kk <= qpos) ? x * sl2 - al2 * static_cast<float>(qpos - kk) : -INFINITY;
      m = fmaxf(m, p[kb][t]);
    }
  }
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  float l = 0.f;
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      p[kb][t] = p[kb][t] == -INFINITY ? 0.f : exp2f(p[kb][t] - m);  // a NaN score stays one
      l += p[kb][t];
    }
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (lane < NQ) {
    ml[wave][lane][0] = m;
    ml[wave][lane][1] = l;
  }

  if constexpr (NQ == 1) {
    float o[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[e] = 0.f;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < EPL; ++e) o[e] = __builtin_fmaf(p[kb][t], static_cast<float>(vr[kb][t][e]), o[e]);
#pragma unroll
    for (int e = 0; e < EPL; ++e) {
      o[e] += __shfl_xor(o[e], 16, 64);
      o[e] += __shfl_xor(o[e], 32, 64);
    }
    if (g == 0)
#pragma unroll
      for (int e = 0; e < EPL; ++e) red[wave][0][EPL * n + e] = o[e];
  } else {
    floatx4 o[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) o[e] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < EPL; ++e)
          o[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(p[kb][t], static_cast<float>(vr[kb][t][e]), o[e], 0, 0, 0);
    if (4 * g < NQ)  // the lane's rows 4 g + i
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < EPL; ++e) red[wave][(4 * g + i) % NQ][EPL * n + e] = o[e][i];
  }
  __syncthreads();

  // sum over the waves, in wave order, each scaled to the chunk's maximum
  for (int e = tid; e < a.n_new * DH; e += 512) {
    const int j = e / DH, col = e % DH;
    float mw[8], M = -INFINITY, L = 0.f, s = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      mw[w] = ml[w][j][0];
      M = fmaxf(M, mw[w]);
    }
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      const float f = mw[w] == -INFINITY ? 0.f : exp2f(mw[w] - M);
      L = __builtin_fmaf(f, ml[w][j][1], L);
      s = __builtin_fmaf(f, red[w][j][col], s);
    }
    if (a.n_chunks == 1) {
      static_cast<bf16*>(a.out)[(static_cast<int64_t>(b) * a.n_new + j) * d + h * DH + col] =
          static_cast<bf16>(s * (1.f / L));
    } else {
      const int64_t pr = ((static_cast<int64_t>(b) * a.H + h) * a.n_chunks + c) * a.n_new + j;
      a.part_o[pr * DH + col] = s;
      if (col == 0) {
        a.part_ml[pr * 2] = M;
        a.part_ml[pr * 2 + 1] = L;
      }
    }
  }
}

// One wave per (sequence, head, query row): merge the chunks, up to 16 at
// once so that their partial rows are all in flight, rescaling what was summed
// before to the new maximum.  13 chunks of 16 rows (one sequence of 778 keys): 3.8 ->
// 3.0 us.
template <int DH>
__global__ __launch_bounds__(256) void ld_attn_decode_combine(DecAttnArgs a) {
  constexpr int CL = DH / 64, U = 16;
  typedef float FRow __attribute__((ext_vector_type(CL)));
  const int lane = threadIdx.x & 63;
  const int r = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (r >= a.n_seq * a.H * a.n_new) return;
  const int b = r / (a.H * a.n_new), h = (r / a.n_new) % a.H, j = r % a.n_new;
  const int64_t p0 = (static_cast<int64_t>(b) * a.H + h) * a.n_chunks * a.n_new + j;  // + c n_new
  const float* po = a.part_o + p0 * DH + lane * CL;
  const float* pm = a.part_ml + p0 * 2;
  float M = -INFINITY, L = 0.f;
  FRow acc = 0.f;
  for (int c0 = 0; c0 < a.n_chunks; c0 += U) {
    FRow v[U];
    float mc[U], lc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {  // past the last chunk: the last again, dropped below
      const int64_t c = static_cast<int64_t>(min(c0 + u, a.n_chunks - 1)) * a.n_new;
      v[u] = *reinterpret_cast<const FRow*>(po + c * DH);
      mc[u] = pm[c * 2];
      lc[u] = pm[c * 2 + 1];
    }
    __builtin_amdgcn_sched_barrier(0);
    float m = M;
#pragma unroll
    for (int u = 0; u < U; ++u) m = fmaxf(m, mc[u]);
    const float keep = M == -INFINITY ? 0.f : exp2f(M - m);
    L *= keep;
    acc *= keep;
    M = m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = c0 + u < a.n_chunks;  // else selected out: 0 times an infinity in v would be NaN
      const float wgt = !in || mc[u] == -INFINITY ? 0.f : exp2f(mc[u] - m);
      L = __builtin_fmaf(wgt, lc[u], L);
      acc += wgt * (in ? v[u] : FRow(0.f));
    }
  }
  acc *= 1.f / L;
  bf16* out = static_cast<bf16*>(a.out) + (static_cast<int64_t>(b) * a.n_new + j) * (static_cast<int64_t>(a.H) * DH) +
              h * DH + lane * CL;
#pragma unroll
  for (int cc = 0; cc < CL; ++cc) out[cc] = static_cast<bf16>(acc[cc]);
}

int grid_for(int64_t items) {
  int64_t g = (items + 255) / 256;
  if (g > 8192) g = 8192;
  if (g < 1) g = 1;
  return static_cast<int>(g);
}

}  // namespace

int skinny_ksplit(int64_t M, int64_t N, int64_t K) {
  (void)M;
  const int64_t tiles = (N + 31) / 32;
  const int64_t chunks = (K + kSkChunk - 1) / kSkChunk;
  int64_t ks = (512 + tiles - 1) / tiles;
  const int64_t most = chunks / kSkWaves;
  if (ks > most) ks = most;
  if (ks > 16) ks = 16;
  if (ks < 1) ks = 1;
  return static_cast<int>(ks);
}

hipError_t launch_gemm_skinny(const SkinnyArgs& g, int ksplit, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  const dim3 grid((g.N + 31) / 32, ksplit);
  if (g.M <= 32)
    hipLaunchKernelGGL(ld_gemm_bf16_skinny<1>, grid, dim3(256), 0, s, g);
  else
    hipLaunchKernelGGL(ld_gemm_bf16_skinny<2>, grid, dim3(256), 0, s, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || ksplit == 1 || g.part_only) return e;
  hipLaunchKernelGGL(ld_skinny_reduce_k, dim3(grid_for(static_cast<int64_t>(g.M) * g.N)), dim3(256), 0,
                     s, g, ksplit);
  return hipGetLastError();
}

hipError_t launch_skinny_reduce_norm(const SkinnyArgs& g, int ksplit, const void* gain, float eps, void* h,
                                     hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  hipLaunchKernelGGL(ld_skinny_reduce_norm_k, dim3(g.M), dim3(1024), 0, s, g, ksplit, static_cast<const bf16*>(gain),
                     eps, static_cast<bf16*>(h));
  return hipGetLastError();
}

hipError_t launch_skinny_reduce_act(const SkinnyArgs& g, int ksplit, int act, int f, void* s_out, hipStream_t s) {
  if (g.M <= 0 || f <= 0) return hipSuccess;
  hipLaunchKernelGGL(ld_skinny_reduce_act_k, dim3(grid_for(static_cast<int64_t>(g.M) * f)), dim3(256), 0, s, g,
                     ksplit, act, f, static_cast<bf16*>(s_out));
  return hipGetLastError();
}

bool dec_gemm_fuses_norm(int64_t M, int64_t K) {
  return M >= 1 && ((M <= kDecGemmMaxM && K <= 2048) || (M <= 16 && K <= 4096));
}

// Rows of the tiles' weights in flight per CU, and the activations' registers,
// set the variant: eight waves with the activations of K <= 2048 (4 chunks
// each) for up to 48 rows, of K <= 4096 (8 chunks) for up to 16, beyond which
// they would spill, one workgroup per CU, each CU taking the same number of
// tiles; else streamed activations, 16 waves while their registers allow.
// Up to 8 rows of K <= 1024 and more than four tiles per CU: four workgroups of
// four waves per CU, the activations of K <= 512 in half the registers.  A tile
// of few chunks costs its latency and its barrier, about 0.9 us a pair of tiles
// whatever K is, which a lone workgroup pays in turn (8 rows, W of 32768 x 64:
// 18.0 -> 10.3 us; 131072 x 64, 512, 1024: 60 -> 19, 61 -> 23, 62 -> 41 us;
// SwiGLU of 11008 and 131072 x 512: 14.2 -> 8.9, 115 -> 42).  Up to 4 tiles per
// CU both are at the launch's 9 to 10 us.
// Streamed, 8 rows without SwiGLU: a fifth chunk in flight where two passes
// then hold all of K, 8192 < K <= 10240 (9664 at 8 rows: 13.2 -> 11.6 us for up
// to 512 columns, 71 -> 59 for 11008, 787 -> 657 for 131072).
// Decoding passes a gain with every activation, ld_gemm_dec (8 rows) either.
template <int MB, int ACT>
hipError_t gemm_dec_t(const SkinnyArgs& g, hipStream_t s) {
  constexpr bool kBare = MB == 1 || ACT == kDecActNone;  // without a gain
  const int tiles = (g.N + kDecCols - 1) / kDecCols;
  auto grid_of = [&](int wgs) {
    const int rounds = (tiles + wgs - 1) / wgs;
    return dim3((tiles + rounds - 1) / rounds);
  };
  if constexpr (MB == 1) {
    if (g.K <= 1024 && tiles > 4 * kDecCus) {
      const dim3 grid = grid_of(4 * kDecCus), block(256);
      if (g.K <= 512 && g.g)
        hipLaunchKernelGGL((ld_gemm_bf16_dec<MB, ACT, true, 4, 2>), grid, block, 0, s, g);
      else if (g.K <= 512)
        hipLaunchKernelGGL((ld_gemm_bf16_dec<MB, ACT, false, 4, 2>), grid, block, 0, s, g);
      else if (g.g)
        hipLaunchKernelGGL((ld_gemm_bf16_dec<MB, ACT, true, 4, 4>), grid, block, 0, s, g);
      else
        hipLaunchKernelGGL((ld_gemm_bf16_dec<MB, ACT, false, 4, 4>), grid, block, 0, s, g);
      return hipGetLastError();
    }
  }
  const dim3 block(512), grid = grid_of(kDecCus);
  if (dec_gemm_fuses_norm(g.M, g.K)) {
    if (g.K <= 2048) {
      if (g.g)
        hipLaunchKernelGGL((ld_gemm_bf16_dec<MB, ACT, true, 8, 4>), grid, block, 0, s, g);
      else if constexpr (kBare)
        hipLaunchKernelGGL((ld_gemm_bf16_dec<MB, ACT, false, 8, 4>), grid, block, 0, s, g);
      else
        return hipErrorInvalidValue;
    } else if constexpr (MB <= 2) {
      if (g.g)
        hipLaunchKernelGGL((ld_gemm_bf16_dec<MB, ACT, true, 8, 8>), grid, block, 0, s, g);
      else if constexpr (kBare)
        hipLaunchKernelGGL((ld_gemm_bf16_dec<MB, ACT, false, 8, 8>), grid, block, 0, s, g);
      else
        return hipErrorInvalidValue;
    }
  } else if constexpr (kBare) {
    if (g.g) return hipErrorInvalidValue;
    constexpr int NW = MB <= 3 ? 16 : 8, U = MB <= 2 && ACT != kDecActSwiglu ? 4 : 2;
    if constexpr (MB == 1 && U == 4) {
      if (g.K > 2 * 64 * NW * U && g.K <= 2 * 64 * NW * (U + 1)) {
        hipLaunchKernelGGL((ld_gemm_bf16_dec_long<MB, ACT, NW, U + 1>), dim3(tiles), dim3(NW * 64), 0, s, g);
        return hipGetLastError();
      }
    }
    hipLaunchKernelGGL((ld_gemm_bf16_dec_long<MB, ACT, NW, U>), dim3(tiles), dim3(NW * 64), 0, s, g);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int MB>
hipError_t gemm_dec_act(const SkinnyArgs& g, hipStream_t s) {
  if (g.act == kDecActSwiglu) return gemm_dec_t<MB, kDecActSwiglu>(g, s);
  if (g.act == kDecActRelu2) return gemm_dec_t<MB, kDecActRelu2>(g, s);
  return gemm_dec_t<MB, kDecActNone>(g, s);
}

hipError_t launch_gemm_dec(const SkinnyArgs& g, hipStream_t s) {
  if (g.N <= 0) return hipSuccess;
  if (g.M < 1 || g.M > kDecGemmMaxM || g.K < 8 || g.K % 8) return hipErrorInvalidValue;
  const int mb = (g.M + 7) / 8;  // blocks of 8 rows
  return mb <= 1   ? gemm_dec_act<1>(g, s)
         : mb <= 2 ? gemm_dec_act<2>(g, s)
         : mb <= 3 ? gemm_dec_act<3>(g, s)
         : mb <= 4 ? gemm_dec_act<4>(g, s)
                   : gemm_dec_act<6>(g, s);
}

hipError_t launch_kv_store(const KvArgs& a, hipStream_t s) {
  const int64_t items = static_cast<int64_t>(a.n_seq) * a.n * (2ll * a.d / 8);
  if (items == 0) return hipSuccess;
  hipLaunchKernelGGL(ld_kv_store_k, dim3(grid_for(items)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Blocks of 8 keys per wave (1 to 4: chunks of 64 to 256 keys).  Up to 256
// keys: one chunk and no second launch.  Beyond, of 64, 128 and 192 keys what
// costs least: rounds of two workgroups per CU, each its keys and about another
// 64 keys' worth of start and end; at equal cost the largest chunk.  The partial
// rows must fit the scratch, which is sized for kDecMaxRows rows of 256-key
// chunks: 256 keys are for where 192 do not fit.  One row over 778 keys and 16
// heads takes 208 workgroups of 64 keys (64 of 256: 9.2 us, now 4.2); six rows of 8
// sequences over 1506 keys 1024 of 192 (768 of 256: 27.4 us, now 23.3); one row
// of 8 sequences over 2048 keys 1408 of 192 (1024 of 256: 28.5 us, now 25.9).
int dec_attn_blocks(const DecAttnArgs& a) {
  const int64_t nk = static_cast<int64_t>(a.pos) + a.n_new, heads = static_cast<int64_t>(a.n_seq) * a.H;
  const int64_t scratch_rows = (nk + kDecKeys - 1) / kDecKeys * kDecMaxRows;
  if (nk <= kDecKeys) return static_cast<int>((nk + 63) / 64);
  int best = 4;
  int64_t best_cost = INT64_MAX;
  for (int kb = 3; kb >= 1; --kb) {
    const int64_t chunks = (nk + 64 * kb - 1) / (64 * kb);
    if (chunks * a.n_new > scratch_rows) break;
    const int64_t cost = (heads * chunks + 2 * kDecCus - 1) / (2 * kDecCus) * (kb + 1);
    if (cost < best_cost) {
      best = kb;
      best_cost = cost;
    }
  }
  return best;
}

template <int DH, int NQ>
hipError_t attn_decode_t(DecAttnArgs a, hipStream_t s) {
  const int kb = dec_attn_blocks(a);
  a.n_chunks = static_cast<int32_t>((static_cast<int64_t>(a.pos) + a.n_new + 64 * kb - 1) / (64 * kb));
  const dim3 grid(a.n_chunks, a.H, a.n_seq);
  if (kb == 1)
    hipLaunchKernelGGL((ld_attn_decode_bf16<DH, NQ, 1>), grid, dim3(512), 0, s, a);
  else if (kb == 2)
    hipLaunchKernelGGL((ld_attn_decode_bf16<DH, NQ, 2>), grid, dim3(512), 0, s, a);
  else if (kb == 3)
    hipLaunchKernelGGL((ld_attn_decode_bf16<DH, NQ, 3>), grid, dim3(512), 0, s, a);
  else
    hipLaunchKernelGGL((ld_attn_decode_bf16<DH, NQ, 4>), grid, dim3(512), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.n_chunks == 1) return e;
  const int rows = a.n_seq * a.H * a.n_new;
  hipLaunchKernelGGL(ld_attn_decode_combine<DH>, dim3((rows + 3) / 4), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int DH>
hipError_t attn_decode_dh(const DecAttnArgs& a, hipStream_t s) {
  if (a.n_new <= 1) return attn_decode_t<DH, 1>(a, s);
  if (a.n_new <= 4) return attn_decode_t<DH, 4>(a, s);
  return attn_decode_t<DH, 8>(a, s);
}

hipError_t launch_attn_decode(const DecAttnArgs& a, hipStream_t s) {
  return a.dh == 128 ? attn_decode_dh<128>(a, s) : attn_decode_dh<64>(a, s);
}

}  // namespace ld
