// GEMM kernels: C[m, n] = (R ? R[m, n] : 0) + alpha * sum_k A(m, k) B(n, k).
//
// bf16 (gfx950 MFMA, float32 accumulation), two kinds:
//   the ring kernels (ld_gemm_bf16_*_256, _128; "big" below): 256 x 256 or 128 x
//   256 tiles, operands fetched straight into an LDS ring, fused epilogues;
//   nearly every GEMM.  Described where they start.
//   the 128x128 kernels (ld_gemm_bf16_nt, _nn, _tn, _tt): for operands or widths
//   the ring kernels do not take, and short products over a ragged edge
//   (gemm_prefers_small).  K step 64, four waves each owning a 64x64 quarter (2x2
//   blocks of v_mfma_f32_32x32x16_bf16).  Both operands are staged in LDS as
//   [row][k] with k contiguous so every MFMA fragment is one 16-byte LDS read; an
//   operand whose k is not contiguous in HBM is transposed on its way: each
//   thread loads four k-rows of eight consecutive m/n values (16-byte coalesced
//   loads) and writes eight 8-byte [m][k0..k0+3] pieces.  LDS is double buffered
//   and the next tile's global loads are issued before the current tile's MFMAs,
//   one barrier per K step.
//
// The row count (forward and input-gradient GEMMs) or the reduction length
// (weight-gradient GEMMs) can be read from a device kept count, so the grid is
// sized for the whole batch and tiles past the kept rows exit at once.
//
// fp32 (the fp32 configuration only): SIMT kernels, ld_gemm_f32_vec_k with 64x64
// or 32x32 tiles, 16-byte loads and double-buffered LDS, and ld_gemm_f32_k with
// 64x64 tiles for unaligned or very short operands (f32_vec).
#include <algorithm>
#include <functional>
#include <initializer_list>
#include <queue>
#include <utility>
#include <type_traits>
#include <vector>

#include "gemm_extent.h"
#include "ld_internal.h"

namespace ld {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int BM = 128, BN = 128, BK = 64, LDK = BK + 8;  // LDS row pitch (bf16)
constexpr int kTileElems = BM * LDK;

__device__ __forceinline__ int64_t map_row(const RowMap& m, int64_t row) {
  if (!m.idx) return row;
  return static_cast<int64_t>(m.idx[row / m.S]) * m.S + row % m.S;
}

__device__ __forceinline__ void resolve_counts(const GemmArgs& g, int& M, int& K) {
  M = g.M;
  K = g.K;
  if (g.dev_count) {
    const int c = *g.dev_count * g.count_mult;
    if (g.count_dim == 0)
      M = c;
    else
      K = c;
  }
}

// ---- operand staging -------------------------------------------------------

// k-contiguous operand X[r * ld + k]: 128 rows x 64 k = 1024 chunks of 8.
struct KRegs {
  uint4 v[4];
};
__device__ __forceinline__ void load_kc(KRegs& t, const bf16* X, int64_t ld, int r0, int R, int k0,
                                        int K, int tid) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int chunk = p * 256 + tid;
    const int row = chunk >> 3, kc = (chunk & 7) * 8;
    const int gr = r0 + row, gk = k0 + kc;
    if (gr < R && gk < K)
      t.v[p] = *reinterpret_cast<const uint4*>(X + static_cast<int64_t>(gr) * ld + gk);
    else
      t.v[p] = make_uint4(0, 0, 0, 0);
  }
}
__device__ __forceinline__ void store_kc(const KRegs& t, bf16* lds, int tid) {
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int chunk = p * 256 + tid;
    const int row = chunk >> 3, kc = (chunk & 7) * 8;
    *reinterpret_cast<uint4*>(lds + row * LDK + kc) = t.v[p];
  }
}

// mn-contiguous operand X[k * ld + r]: thread loads k-rows kg..kg+3 of the
// eight r values rc..rc+7 and writes them transposed.
__device__ __forceinline__ void load_mc(KRegs& t, const bf16* X, int64_t ld, int r0, int R, int k0,
                                        int K, int tid) {
  const int rc = (tid & 15) * 8, kg = (tid >> 4) * 4;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const int gk = k0 + kg + kk, gr = r0 + rc;
    if (gk < K && gr < R)
      t.v[kk] = *reinterpret_cast<const uint4*>(X + static_cast<int64_t>(gk) * ld + gr);
    else
      t.v[kk] = make_uint4(0, 0, 0, 0);
  }
}
__device__ __forceinline__ uint32_t half_of(const uint4& v, int i) {
  const uint32_t w = (i >> 1) == 0 ? v.x : (i >> 1) == 1 ? v.y : (i >> 1) == 2 ? v.z : v.w;
  return (i & 1) ? (w >> 16) : (w & 0xffffu);
}
__device__ __forceinline__ void store_mc(const KRegs& t, bf16* lds, int tid) {
  const int rc = (tid & 15) * 8, kg = (tid >> 4) * 4;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    uint2 o;
    o.x = half_of(t.v[0], i) | (half_of(t.v[1], i) << 16);
    o.y = half_of(t.v[2], i) | (half_of(t.v[3], i) << 16);
    *reinterpret_cast<uint2*>(lds + (rc + i) * LDK + kg) = o;
  }
}

template <bool KC>
__device__ __forceinline__ void load_op(KRegs& t, const bf16* X, int64_t ld, int r0, int R, int k0,
                                        int K, int tid) {
  if constexpr (KC)
    load_kc(t, X, ld, r0, R, k0, K, tid);
  else
    load_mc(t, X, ld, r0, R, k0, K, tid);
}
template <bool KC>
__device__ __forceinline__ void store_op(const KRegs& t, bf16* lds, int tid) {
  if constexpr (KC)
    store_kc(t, lds, tid);
  else
    store_mc(t, lds, tid);
}

// ---- epilogue -------------------------------------------------------------
// 32x32 accumulator layout: lane l, register v holds row
// 8*(v/4) + 4*(l/32) + v%4 and column l%32 of the block.
__device__ __forceinline__ void epilogue_store(const GemmArgs& g, float alpha, int row, int col,
                                               float acc, int M) {
  if (row >= M || col >= g.N) return;
  float val = alpha * acc;
  const int64_t orow = map_row(g.out_map, row);
  if (g.R) {
    const int64_t rrow = g.r_mapped ? orow : row;
    if (g.r_f32)
      val += static_cast<const float*>(g.R)[rrow * g.ldr + col];
    else
      val += static_cast<float>(static_cast<const bf16*>(g.R)[rrow * g.ldr + col]);
  }
  if (g.c_f32)
    static_cast<float*>(g.C)[orow * g.ldc + col] = val;
  else
    static_cast<bf16*>(g.C)[orow * g.ldc + col] = static_cast<bf16>(val);
}

template <bool AK, bool BKC>
__device__ __forceinline__ void gemm_bf16_body(const GemmArgs& g) {
  extern __shared__ __align__(16) bf16 smem[];
  bf16* As = smem;                  // [2][BM][LDK]
  bf16* Bs = smem + 2 * kTileElems;  // [2][BN][LDK]
  int M, K;
  resolve_counts(g, M, K);
  const int tiles_n = (g.N + BN - 1) / BN;
  const int tm = blockIdx.x / tiles_n, tn = blockIdx.x % tiles_n;
  const int m0 = tm * BM, n0 = tn * BN;
  if (m0 >= M) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const bf16* A = static_cast<const bf16*>(g.A);
  const bf16* B = static_cast<const bf16*>(g.B);

  floatx16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int nk = (K + BK - 1) / BK;
  if (nk > 0) {
    KRegs ra, rb;
    load_op<AK>(ra, A, g.lda, m0, M, 0, K, tid);
    load_op<BKC>(rb, B, g.ldb, n0, g.N, 0, K, tid);
    store_op<AK>(ra, As, tid);
    store_op<BKC>(rb, Bs, tid);
    __syncthreads();
    const int lrow = lane & 31, lk = (lane >> 5) * 8;
    for (int kt = 0; kt < nk; ++kt) {
      const int buf = kt & 1;
      if (kt + 1 < nk) {
        load_op<AK>(ra, A, g.lda, m0, M, (kt + 1) * BK, K, tid);
        load_op<BKC>(rb, B, g.ldb, n0, g.N, (kt + 1) * BK, K, tid);
      }
      const bf16* as = As + buf * kTileElems;
      const bf16* bs = Bs + buf * kTileElems;
#pragma unroll
      for (int ks = 0; ks < BK / 16; ++ks) {
        bf16x8 af[2], bfr[2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
          af[i] = *reinterpret_cast<const bf16x8*>(as + (wm * 64 + i * 32 + lrow) * LDK + ks * 16 + lk);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          bfr[j] = *reinterpret_cast<const bf16x8*>(bs + (wn * 64 + j * 32 + lrow) * LDK + ks * 16 + lk);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
      }
      if (kt + 1 < nk) {
        store_op<AK>(ra, As + (buf ^ 1) * kTileElems, tid);
        store_op<BKC>(rb, Bs + (buf ^ 1) * kTileElems, tid);
      }
      __syncthreads();
    }
  }
  const float alpha = g.alpha * (g.alpha_dev ? *g.alpha_dev : 1.f);
  const int half = lane >> 5, col_l = lane & 31;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int row = m0 + wm * 64 + i * 32 + 8 * (v >> 2) + 4 * half + (v & 3);
        const int col = n0 + wn * 64 + j * 32 + col_l;
        epilogue_store(g, alpha, row, col, acc[i][j][v], M);
      }
}

__global__ __launch_bounds__(256) void ld_gemm_bf16_nt(GemmArgs g) { gemm_bf16_body<true, true>(g); }
__global__ __launch_bounds__(256) void ld_gemm_bf16_nn(GemmArgs g) { gemm_bf16_body<true, false>(g); }
__global__ __launch_bounds__(256) void ld_gemm_bf16_tn(GemmArgs g) { gemm_bf16_body<false, false>(g); }
__global__ __launch_bounds__(256) void ld_gemm_bf16_tt(GemmArgs g) { gemm_bf16_body<false, true>(g); }

// ---- fp32 SIMT ------------------------------------------------------------

constexpr int FT = 64, FK = 16;

template <bool AK, bool BKC>
__global__ __launch_bounds__(256) void ld_gemm_f32_k(GemmArgs g) {
  __shared__ float As[FK][FT + 4], Bs[FK][FT + 4];
  int M, K;
  resolve_counts(g, M, K);
  const int tiles_n = (g.N + FT - 1) / FT;
  const int m0 = (blockIdx.x / tiles_n) * FT, n0 = (blockIdx.x % tiles_n) * FT;
  if (m0 >= M) return;
  const float* A = static_cast<const float*>(g.A);
  const float* B = static_cast<const float*>(g.B);
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += FK) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int id = e * 256 + tid;
      int mm, kk;
      if (AK) { mm = id / FK; kk = id % FK; } else { kk = id / FT; mm = id % FT; }
      const int gm = m0 + mm, gk = k0 + kk;
      float v = 0.f;
      if (gm < M && gk < K) v = AK ? A[static_cast<int64_t>(gm) * g.lda + gk] : A[static_cast<int64_t>(gk) * g.lda + gm];
      As[kk][mm] = v;
      int nn;
      if (BKC) { nn = id / FK; kk = id % FK; } else { kk = id / FT; nn = id % FT; }
      const int gn = n0 + nn, gk2 = k0 + kk;
      float w = 0.f;
      if (gn < g.N && gk2 < K) w = BKC ? B[static_cast<int64_t>(gn) * g.ldb + gk2] : B[static_cast<int64_t>(gk2) * g.ldb + gn];
      Bs[kk][nn] = w;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < FK; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) a[r] = As[kk][ty * 4 + r];
#pragma unroll
      for (int c = 0; c < 4; ++c) b[c] = Bs[kk][tx * 4 + c];
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = __builtin_fmaf(a[r], b[c], acc[r][c]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int row = m0 + ty * 4 + r, col = n0 + tx * 4 + c;
      if (row >= M || col >= g.N) continue;
      float val = g.alpha * (g.alpha_dev ? *g.alpha_dev : 1.f) * acc[r][c];
      const int64_t orow = map_row(g.out_map, row);
      if (g.R) val += static_cast<const float*>(g.R)[(g.r_mapped ? orow : row) * g.ldr + col];
      static_cast<float*>(g.C)[orow * g.ldc + col] = val;
    }
}

// The same product (each output one chain of fused multiply-adds over k, the
// same bits) for operands of 16-byte aligned rows: TS x TS tiles, k in tiles of
// 32, 16-byte loads two k tiles ahead of the arithmetic and double-buffered
// LDS, one barrier per k tile.  At the sizes of the float32 configurations a
// GEMM is a handful of tiles, and its time the latency of its chain of k tiles:
// the kernel above, whose loads each stand in a branch of their own and are
// waited for one by one, takes 40 us for 192 x 64 x 256 and this one 6.
constexpr int FKV = 32;

template <bool AK, bool BKC, int TS>
__global__ __launch_bounds__(256) void ld_gemm_f32_vec_k(GemmArgs g) {
  constexpr int NV = TS * FKV / 4 / 256;  // float4 per thread, operand and k tile
  constexpr int TT = TS / 16;             // outputs per thread: TT x TT
  __shared__ __align__(16) float As[2][FKV][TS + 4], Bs[2][FKV][TS + 4];
  int M, K;
  resolve_counts(g, M, K);
  const int N = g.N;
  const int tiles_n = (N + TS - 1) / TS;
  const int m0 = (blockIdx.x / tiles_n) * TS, n0 = (blockIdx.x % tiles_n) * TS;
  if (m0 >= M) return;
  const float* A = static_cast<const float*>(g.A);
  const float* B = static_cast<const float*>(g.B);
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int nk = (K + FKV - 1) / FKV;
  struct Regs {
    float4 a[NV], b[NV];
  };
  // Rows past M (N) repeat the last, k past K the first: no branch around a
  // load; k past K is zeroed on its way into LDS.
  auto load = [&](Regs& r, int kt) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int id = v * 256 + tid;
      const int kc = kt * FKV + 4 * (id % (FKV / 4)), rc = id / (FKV / 4);  // k-contiguous: row rc, 4 k
      const int km = kt * FKV + id / (TS / 4), rm = 4 * (id % (TS / 4));    // else: k row km, 4 columns
      if (AK)
        r.a[v] = *reinterpret_cast<const float4*>(A + static_cast<int64_t>(min(m0 + rc, M - 1)) * g.lda + (kc < K ? kc : 0));
      else
        r.a[v] = *reinterpret_cast<const float4*>(A + static_cast<int64_t>(km < K ? km : 0) * g.lda + min(m0 + rm, M - 4));
      if (BKC)
        r.b[v] = *reinterpret_cast<const float4*>(B + static_cast<int64_t>(min(n0 + rc, N - 1)) * g.ldb + (kc < K ? kc : 0));
      else
        r.b[v] = *reinterpret_cast<const float4*>(B + static_cast<int64_t>(km < K ? km : 0) * g.ldb + min(n0 + rm, N - 4));
    }
  };
  auto store = [&](const Regs& r, int kt) {
    const int buf = kt & 1;
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      const int id = v * 256 + tid;
      const int kc = 4 * (id % (FKV / 4)), rc = id / (FKV / 4);
      const int km = id / (TS / 4), rm = 4 * (id % (TS / 4));
      const bool okc = kt * FKV + kc < K, okm = kt * FKV + km < K;
      auto put = [&](float (&L)[FKV][TS + 4], float4 x, bool kcontig) {
        const bool ok = kcontig ? okc : okm;
        x = make_float4(ok ? x.x : 0.f, ok ? x.y : 0.f, ok ? x.z : 0.f, ok ? x.w : 0.f);
        if (kcontig) {
          L[kc][rc] = x.x;
          L[kc + 1][rc] = x.y;
          L[kc + 2][rc] = x.z;
          L[kc + 3][rc] = x.w;
        } else {
          *reinterpret_cast<float4*>(&L[km][rm]) = x;
        }
      };
      put(As[buf], r.a[v], AK);
      put(Bs[buf], r.b[v], BKC);
    }
  };
  float acc[TT][TT] = {};
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < FKV; ++kk) {
      float a[TT], b[TT];
#pragma unroll
      for (int r = 0; r < TT; ++r) a[r] = As[buf][kk][ty * TT + r];
#pragma unroll
      for (int c = 0; c < TT; ++c) b[c] = Bs[buf][kk][tx * TT + c];
#pragma unroll
      for (int r = 0; r < TT; ++r)
#pragma unroll
        for (int c = 0; c < TT; ++c) acc[r][c] = __builtin_fmaf(a[r], b[c], acc[r][c]);
    }
  };
  if (nk > 0) {
    Regs r0, r1;
    load(r0, 0);
    load(r1, 1);  // a k tile past the end reads the operands' first rows
    for (int kt = 0; kt < nk; kt += 2) {
      store(r0, kt);
      __syncthreads();
      load(r0, kt + 2);
      compute(0);
      if (kt + 1 < nk) {
        store(r1, kt + 1);
        __syncthreads();
        load(r1, kt + 3);
        compute(1);
      }
    }
  }
  const float alpha = g.alpha * (g.alpha_dev ? *g.alpha_dev : 1.f);
#pragma unroll
  for (int r = 0; r < TT; ++r)
#pragma unroll
    for (int c = 0; c < TT; ++c) {
      const int row = m0 + ty * TT + r, col = n0 + tx * TT + c;
      if (row >= M || col >= N) continue;
      float val = alpha * acc[r][c];
      const int64_t orow = map_row(g.out_map, row);
      if (g.R) val += static_cast<const float*>(g.R)[(g.r_mapped ? orow : row) * g.ldr + col];
      static_cast<float*>(g.C)[orow * g.ldc + col] = val;
    }
}

constexpr size_t kGemmLds = 4 * kTileElems * sizeof(bf16);

// ===================================================================== big
// 256x256 workgroup tile, eight waves in a 4x2 grid each owning 64x128 (4x8
// blocks of v_mfma_f32_16x16x32_bf16, 128 fp32 accumulators per lane), k
// walked in steps of 64.
//
// What bounds it: on random data the chip lowers its clock under sustained
// MFMA load (the same kernel runs ~20% faster on zeros), so energy counts as
// much as stalls.  Two waves per SIMD instead of one wave of 128x128: when a
// wave stalls issuing a load or waits at its epilogue, the other one's MFMAs
// go on; that outweighs the half more LDS reads.  16x16x32 rather than
// 32x32x16 MFMAs: half the accumulator traffic per product, 2-4% faster at
// the clock limit.  Against the four-wave kernel with 32x32x16 MFMAs that
// this replaced, same box, random data: NT 8192^3 802 -> 727 us (1512
// TFLOP/s), 14336 x 11008 x 2048 533 -> 472 us (1369 TFLOP/s); NN 14336 x
// 2048 x 11008 516 -> 485 us; TN 2048 x 2048 x 14336 116 -> 108 us.
//
// Operand tiles go from global memory straight into LDS: buffer loads with an
// LDS destination, so no register staging and no LDS write instructions.
// Such a load writes the 16 bytes of lane i at LDS offset 16*i from a
// wave-uniform base, so the LDS layout is set by which global chunk each lane
// fetches.  The ring (the whole 160 KB of LDS) holds three slots of A and two
// of B, each one k step of 256 rows or columns (32 KB):
//   mn-contiguous operand: [64 k][256 mn] as in memory, chunks XOR-swizzled
//     by k; a load instruction fetches two whole 512-byte k rows.  A fragment
//     is two transposing reads (ds_read_b64_tr_b16: in each group of 16
//     lanes, lane j receives element j%4 of the four-element rows read by
//     lanes j/4, j/4+4, j/4+8 and j/4+12, so 16 lanes reading rows k..k+3 at
//     mn offsets 0, 4, 8, 12 give lane j the values k..k+3 at mn j).
//   k-contiguous operand: [256 rows][64 k], so a load instruction fetches 8
//     rows as whole 128-byte lines.  The 16-byte chunks of a row are
//     XOR-swizzled by the row; a fragment is one 16-byte read per lane.
// Rows past the operand's end, and k chunks past the split's end, are
// fetched from an offset outside the buffer descriptor's range and land in
// LDS as zeros.  The loads are issued as inline assembly (ld_internal.h),
// so the compiler does not track them; the kernel waits for them itself
// (s_waitcnt vmcnt) before the barriers.
//
// A k step is four quarters h of 16 MFMAs per wave: k-substep (32) h / 2 and
// four of the eight B blocks.  Each quarter reads the fragments of the next
// one, so no MFMA waits on a recent LDS read.  The one barrier of step t
// stands before its last quarter, where every wave has read all of step t's
// fragments and step t+1 has landed; after it B's slot of step t takes step
// t+2 (four loads spread over the last quarter) and A's slot of step t-1 takes
// step t+2 (spread over the next quarter).  Spread evenly and issued right
// after the barrier the loads have most of a step to land: two quarters later
// they cost 5% (NT 8192^3), in a burst 2-4%.
//
// The MFMA is issued as B x A so each lane ends with 4 consecutive output
// columns of one row.  Tiles are ordered XCD-aware: consecutive workgroup ids
// go to different XCDs, so ids are remapped to give each XCD a contiguous
// range of tiles, walked in groups of 4 or 8 tile-rows for L2 reuse.  Split-K
// (grid.y) writes fp32 partials that a second kernel sums in split order.

constexpr int GB = 256, GK = 64;
constexpr int kBigThreads = 512;        // eight waves
constexpr int kSlot = GB * GK;          // elements of a k step of 256 rows or columns
constexpr int kLoads = 4;               // load instructions per wave per 256-row slot
constexpr int kWaitVm0 = 0x0F70;        // s_waitcnt vmcnt(0), the other counters untouched
constexpr int kRingElems = 5 * kSlot;   // 160 KB
constexpr uint32_t kOob = kDmaOob;
constexpr int64_t kBigMaxSpan = kDmaMaxSpan;
static_assert(kRingElems * 2 <= 160 * 1024, "the ring fits the LDS");

// The tile of BM rows (256 or 128) x 256 columns and its waves' parts: eight
// waves in a (BM / 64) x NWN grid, each 64 rows x WC columns.  Three slots of A
// and NSB of B fit the ring.
template <int BM>
struct BigShape {
  static constexpr int NWN = BM == 256 ? 2 : 4, WC = 256 / NWN;
  static constexpr int NJ = WC / 16;               // 16-column blocks per wave
  static constexpr int SlotA = BM * GK, LoadsA = kLoads * BM / 256;
  static constexpr int NSA = 3, NSB = BM == 256 ? 2 : 3;
  static constexpr int Elems = NSA * SlotA + NSB * kSlot;
  // epilogue staging: WC + 4 elements per row; RPI rows per load or store of
  // 4 floats per lane
  static constexpr int Pitch = WC + 4, RPI = 256 / WC, NIT = 32 / RPI;
};
static_assert(BigShape<256>::Elems <= kRingElems && BigShape<128>::Elems <= kRingElems, "the slots fit the ring");
static_assert(kRingElems * 2 >= 8 * 32 * BigShape<256>::Pitch * 4, "epilogue staging fits the ring");

typedef short v4s __attribute__((ext_vector_type(4)));
typedef dma_rsrc v4i;
#define LD_LDS(T, p) ((__attribute__((address_space(3))) T*)(p))

// k-contiguous slot: element (row, k) of [256][64].  The chunk
// swizzle uses row bits 1-3: of 16 lanes reading one chunk of 16
// consecutive rows, the two rows of each pair sit 128 bytes apart and the 8
// pairs on 8 different chunks, so all 16 hit different 16-byte bank groups;
// moving by a multiple of 16 rows is a plain offset.
__device__ __forceinline__ int kc_swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int swz_off(int row, int k) {
  return row * GK + ((((k >> 3) ^ kc_swz(row)) << 3) | (k & 7));
}

// mn-contiguous slot: element (k, m) of [64][256].  The swizzle puts the 4 k
// rows a 16-lane transposing read touches (32 bytes each) on 4 different
// 64-byte bank groups, and rows k and k+8 on different halves; it depends on
// k bits 0, 1 and 3 only, so k steps of 4 and 16 are plain offsets.
__device__ __forceinline__ int mc_swz(int k) { return ((k & 3) << 2) | (((k >> 3) & 1) << 1); }
__device__ __forceinline__ int mc_off(int k, int m) {
  return k * GB + ((((m >> 3) ^ mc_swz(k)) << 3) | (m & 7));
}

// Per-lane constants of one operand's tile loads and fragment reads.
template <bool KC>
struct OpLanes {
  uint32_t ld_off;  // byte offset of the lane's first 16-byte chunk
  int kchunk;       // k-contiguous: k offset of the lane's chunk in the slot
  int frag[8];      // element offsets of fragment reads: per k-substep (KC) or block (MC)
};

// `r`: the first of the wave's fragment rows.
template <bool KC>
__device__ __forceinline__ OpLanes<KC> op_lanes(int64_t ld, int lane, int wave, int r) {
  OpLanes<KC> o;
  if constexpr (KC) {
    // load instruction p fills slot rows 64p + 8 wave .. +7, lane -> row
    // + lane/8, physical chunk lane%8; the swizzle is the same for every p
    const int row = wave * 8 + (lane >> 3);
    o.kchunk = ((lane & 7) ^ kc_swz(row)) << 3;
    o.ld_off = static_cast<uint32_t>((static_cast<int64_t>(row) * ld + o.kchunk) * 2);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) o.frag[ks] = swz_off(r + (lane & 15), ks * 32 + (lane >> 4) * 8);
  } else {
    // load instruction p fills k rows 16p + 2*wave + lane/32, physical chunk
    // lane%32; the swizzle is the same for every p
    const int kr = 2 * wave + (lane >> 5);
    const int m = ((lane & 31) ^ mc_swz(kr)) << 3;
    o.ld_off = static_cast<uint32_t>((static_cast<int64_t>(kr) * ld + m) * 2);
    o.kchunk = 0;
    // transposing reads: lane reads k row kl, 4 elements from mn ml
    const int kl = (lane >> 4) * 8 + ((lane >> 2) & 3);
    const int ml = 4 * (lane & 3);
#pragma unroll
    for (int i = 0; i < 8; ++i) o.frag[i] = mc_off(kl, r + ml + 16 * i);
  }
  return o;
}

// Load instruction p (0-3) of operand X's rows r0.. (k-contiguous: slot rows
// 64p..64p+63; mn-contiguous: k rows 16p..16p+15) of the k step at k0 into the
// slot at `lds`, 16 bytes per lane.  Columns past the end of an mn-contiguous
// row read the next row's, or zeros past the operand's last element; they only
// reach outputs that are never stored.  A k tail of a k-contiguous operand is
// fetched out of range (zeros), as is everything of a step that starts at or
// past K.  `extent`: mc_extent of the split's k rows (mn-contiguous only).
template <bool KC>
__device__ __forceinline__ void tile_part(bf16* lds, const OpLanes<KC>& o, const bf16* X, int64_t ld, int64_t extent,
                                          int r0, int R, int k0, int K, int wave, int p) {
  if constexpr (KC) {
    const v4i rs = dma_make_rsrc(X + static_cast<int64_t>(r0) * ld, kc_extent(R, r0, ld));
    const uint32_t u = static_cast<uint32_t>((static_cast<int64_t>(p) * 64 * ld + k0) * 2);
    const uint32_t off = k0 + o.kchunk < K ? o.ld_off + u : kOob;
    dma16(rs, lds + (p * 8 + wave) * 512, off);
  } else {
    const int64_t at = mc_offset(k0, ld);
    const v4i rs = dma_make_rsrc(reinterpret_cast<const char*>(X) + at, extent - at);
    const uint32_t u = static_cast<uint32_t>((static_cast<int64_t>(p) * 16 * ld + r0) * 2);
    dma16(rs, lds + (p * 8 + wave) * 512, o.ld_off + u);
  }
}

// B slot of the fused SwiGLU forward: each wave's WC columns pair WC / 2 gate
// rows of W_gate_up [2f, K] with their up rows.  For WC = 128 the slot's 64-row
// block p holds gate rows (p even) or up rows (p odd) tn*128 + (p/2)*64 .. +63;
// for WC = 64 gate rows tn*128 + 32p .. +31, then the up rows.  Load
// instruction p fills rows 8 wave .. +7 of block p.
template <int WC>
__device__ __forceinline__ void tile_part_glu(bf16* lds, const OpLanes<true>& o, const bf16* W, int64_t ld,
                                              int tn, int f, int k0, int K, int wave, int p) {
  // W row of the block's row 0 (the lane's offset adds 8 wave + lane / 8)
  const int64_t rbase = WC == 128
                            ? ((p & 1) ? f : 0) + static_cast<int64_t>(tn) * 128 + (p >> 1) * 64
                            : (wave >= 4 ? f - 32 : 0) + static_cast<int64_t>(tn) * 128 + p * 32;
  const v4i rs = dma_make_rsrc(W + rbase * ld, 64 * ld * 2);
  const uint32_t off = k0 + o.kchunk < K ? o.ld_off + static_cast<uint32_t>(k0 * 2) : kOob;
  dma16(rs, lds + (p * 8 + wave) * 512, off);
}

// Fragment of 16-row block i of the wave's rows for k-substep ks (32) of the
// slot at t: the lane's MFMA row is r + 16 i + lane % 16 (r as given to
// op_lanes), its 8 k values start at ks*32 + (lane/16)*8.  Only the per-lane
// offset is a register; the rest is a constant offset of the LDS instruction.
template <bool KC>
__device__ __forceinline__ bf16x8 frag(const bf16* t, const OpLanes<KC>& o, int i, int ks) {
  if constexpr (KC) {
    return *reinterpret_cast<const bf16x8*>(t + 16 * i * GK + o.frag[ks]);
  } else {
    const bf16* p = t + o.frag[i] + ks * 32 * GB;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LD_LDS(v4s, p));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LD_LDS(v4s, p + 4 * GB));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
}

// Tile of workgroup `pid` among the n_valid = tiles_m * tiles_n tiles that
// hold rows (tiles_m counts only tile rows below the kept count), or false
// when the workgroup has none.  Workgroup ids are dealt to the 8 XCDs in
// turn (id % 8), so XCD x is given its own contiguous, balanced range of
// n_valid / 8 (+1) tiles: the tiles of rows past the kept count are not
// piled onto the last XCDs, and consecutive tiles share an XCD's L2.  Within
// a range, tiles go in groups of tile rows, column by column: groups of 8, or
// of 4 when the matrix has at most 8 tile columns, so that the 32 tiles an XCD
// works on at a time cover every column of B (NN 14336 x 2048 x 11008 with
// groups of 8 499 us, of 4 483 us; with 32 columns 8 is 1-2% better).  The grid has
// at least as many ids per XCD as the largest range (it is sized for every
// row), so every tile is taken.
__device__ __forceinline__ bool tile_coords(int pid, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int n_valid = tiles_m * tiles_n;
  const int x = pid & 7, li = pid >> 3;
  const int base = n_valid >> 3, rem = n_valid & 7;
  if (li >= base + (x < rem ? 1 : 0)) return false;
  const int t = x * base + min(x, rem) + li;
  const int G = tiles_n <= 8 ? 4 : 8;
  const int group = G * tiles_n;
  const int first_m = (t / group) * G;
  const int gsz = min(tiles_m - first_m, G);
  const int in = t % group;
  tm = first_m + in % gsz;
  tn = in / gsz;
  return true;
}

// Loads and stores of outputs and residuals, 8 or 16 bytes at the alignment of
// their elements: gradients may be views into a flat buffer, at any offset.
// (gfx950 takes such addresses in one instruction; the types say so to the
// compiler.)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x4u __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4u __attribute__((ext_vector_type(4), aligned(2)));

__device__ __forceinline__ float4 load_f4(const float* p) {
  const f32x4u v = *reinterpret_cast<const f32x4u*>(p);
  return make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void store_f4(float* p, float4 v) {
  *reinterpret_cast<f32x4u*>(p) = f32x4u{v.x, v.y, v.z, v.w};
}
__device__ __forceinline__ uint2 load_b4(const bf16* p) {
  return __builtin_bit_cast(uint2, *reinterpret_cast<const bf16x4u*>(p));
}
__device__ __forceinline__ void store_b4(bf16* p, float a, float b, float c, float d) {
  *reinterpret_cast<bf16x4u*>(p) = bf16x4u{static_cast<bf16>(a), static_cast<bf16>(b), static_cast<bf16>(c), static_cast<bf16>(d)};
}
__device__ __forceinline__ void store_b8(bf16* p, uint4 v) {
  *reinterpret_cast<u32x4u*>(p) = u32x4u{v.x, v.y, v.z, v.w};
}

// Epilogue of one staged 32-row block row: the lane's rows are r0 + RPI it
// (it < NIT), its 4 columns n..n+3; the staged values (alpha applied) sit at
// stage[(RPI it + sub) * Pitch + c], sub the lane's row of each RPI.
//
// Full block row (every row < M, every column < N): the staged values, row
// map entries and residual values of half the rows are requested before their
// first store, so their latencies overlap, and no branch splits the rows.
template <class SH>
__device__ __forceinline__ void epilogue_rows_full(const GemmArgs& g, float* part, const float* stage,
                                                   int r0, int sub, int c, int n, int q_last) {
  constexpr int NR = 8, RPI = SH::RPI;  // rows in hand (16 would spill next to the accumulators)
  // output row = idx[r / S] * S + r % S; for S >= 32 the 32 rows span at most
  // two sequences
  const int S = g.out_map.S;
  int q0 = 0, rem0 = 0, s0 = 0, s1 = 0;
  if (!part && g.out_map.idx) {
    q0 = r0 / S;
    rem0 = r0 - q0 * S;
    if (S >= 32) {
      s0 = g.out_map.idx[q0];
      s1 = g.out_map.idx[min(q0 + 1, q_last)];
    }
  }
#pragma unroll
  for (int h = 0; h < SH::NIT / NR; ++h) {
    float4 v[NR];
#pragma unroll
    for (int it = 0; it < NR; ++it)
      v[it] = *reinterpret_cast<const float4*>(stage + (RPI * (NR * h + it) + sub) * SH::Pitch + c);
    if (part) {
#pragma unroll
      for (int it = 0; it < NR; ++it)
        *reinterpret_cast<float4*>(part + static_cast<int64_t>(r0 + RPI * (NR * h + it)) * g.N + n) = v[it];
      continue;
    }
    int32_t orow[NR];
#pragma unroll
    for (int it = 0; it < NR; ++it) {
      const int r = r0 + RPI * (NR * h + it);
      orow[it] = r;
      if (g.out_map.idx) {
        if (S >= 32) {
          const int rr = rem0 + RPI * (NR * h + it);
          orow[it] = rr >= S ? s1 * S + (rr - S) : s0 * S + rr;
        } else {
          const int q = r / S;
          orow[it] = g.out_map.idx[q] * S + (r - q * S);
        }
      }
    }
    if (g.R && g.r_f32) {  // float32 residual (the residual streams)
      const float* R = static_cast<const float*>(g.R);
      float4 rv[NR];
#pragma unroll
      for (int it = 0; it < NR; ++it) {
        const int64_t rrow = g.r_mapped ? orow[it] : r0 + RPI * (NR * h + it);
        rv[it] = load_f4(R + rrow * g.ldr + n);
      }
#pragma unroll
      for (int it = 0; it < NR; ++it) {
        v[it].x += rv[it].x;
        v[it].y += rv[it].y;
        v[it].z += rv[it].z;
        v[it].w += rv[it].w;
      }
    } else if (g.R) {  // bf16 residual
      uint2 rv[NR];
      const bf16* R = static_cast<const bf16*>(g.R);
#pragma unroll
      for (int it = 0; it < NR; ++it) {
        const int64_t rrow = g.r_mapped ? orow[it] : r0 + RPI * (NR * h + it);
        rv[it] = load_b4(R + rrow * g.ldr + n);
      }
#pragma unroll
      for (int it = 0; it < NR; ++it) {
        const bf16* rb = reinterpret_cast<const bf16*>(&rv[it]);
        v[it].x += static_cast<float>(rb[0]);
        v[it].y += static_cast<float>(rb[1]);
        v[it].z += static_cast<float>(rb[2]);
        v[it].w += static_cast<float>(rb[3]);
      }
    }
    if (g.c_f32) {
#pragma unroll
      for (int it = 0; it < NR; ++it)
        store_f4(static_cast<float*>(g.C) + static_cast<int64_t>(orow[it]) * g.ldc + n, v[it]);
    } else {
#pragma unroll
      for (int it = 0; it < NR; ++it)
        store_b4(static_cast<bf16*>(g.C) + static_cast<int64_t>(orow[it]) * g.ldc + n, v[it].x, v[it].y, v[it].z, v[it].w);
    }
  }
}

// Block row with rows past M or columns past N: one row at a time, each
// checked.
template <class SH>
__device__ __forceinline__ void epilogue_rows_edge(const GemmArgs& g, float* part, const float* stage,
                                                   int r0, int sub, int c, int n, int M) {
#pragma unroll 1
  for (int it = 0; it < SH::NIT; ++it) {
    const int m = r0 + SH::RPI * it;
    if (m >= M || n >= g.N) continue;
    float4 v = *reinterpret_cast<const float4*>(stage + (SH::RPI * it + sub) * SH::Pitch + c);
    if (part) {
      *reinterpret_cast<float4*>(part + static_cast<int64_t>(m) * g.N + n) = v;
      continue;
    }
    const int64_t orow = map_row(g.out_map, m);
    if (g.R) {
      const int64_t rrow = g.r_mapped ? orow : m;
      if (g.r_f32) {
        const float4 r = load_f4(static_cast<const float*>(g.R) + rrow * g.ldr + n);
        v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w;
      } else {
        const uint2 r = load_b4(static_cast<const bf16*>(g.R) + rrow * g.ldr + n);
        const bf16* rb = reinterpret_cast<const bf16*>(&r);
        v.x += static_cast<float>(rb[0]); v.y += static_cast<float>(rb[1]);
        v.z += static_cast<float>(rb[2]); v.w += static_cast<float>(rb[3]);
      }
    }
    if (g.c_f32) {
      store_f4(static_cast<float*>(g.C) + orow * g.ldc + n, v);
    } else {
      store_b4(static_cast<bf16*>(g.C) + orow * g.ldc + n, v.x, v.y, v.z, v.w);
    }
  }
}

constexpr int kEpiPlain = 0, kEpiGluFwd = 1, kEpiGluBwd = 2, kEpiRelu2Fwd = 3, kEpiRelu2Bwd = 4, kEpiKv = 5;

__device__ __forceinline__ uint2 pack4_bf16(float a, float b, float c, float d) {
  __attribute__((aligned(8))) bf16 o[4] = {static_cast<bf16>(a), static_cast<bf16>(b), static_cast<bf16>(c),
                                           static_cast<bf16>(d)};
  return *reinterpret_cast<const uint2*>(o);
}

__device__ __forceinline__ float4 unpack4_bf16(uint2 r) {
  const bf16* b = reinterpret_cast<const bf16*>(&r);
  return make_float4(static_cast<float>(b[0]), static_cast<float>(b[1]), static_cast<float>(b[2]),
                     static_cast<float>(b[3]));
}

// Fused SwiGLU backward: the staged gs values (alpha applied; rows r0 + 2 it,
// columns n..n+3 < N = f), kept in float32 (gs is never stored), with u and
// v read from aux, give gu and gv in C columns n and f + n.
__device__ __forceinline__ void glu_bwd_one(const GemmArgs& g, float4 gs, uint2 ur, uint2 vr, int64_t m, int n) {
  const float4 u = unpack4_bf16(ur), v = unpack4_bf16(vr);
  float gu[4], gv[4];
  swiglu_bwd_f(u.x, v.x, gs.x, gu[0], gv[0]);
  swiglu_bwd_f(u.y, v.y, gs.y, gu[1], gv[1]);
  swiglu_bwd_f(u.z, v.z, gs.z, gu[2], gv[2]);
  swiglu_bwd_f(u.w, v.w, gs.w, gu[3], gv[3]);
  bf16* C = static_cast<bf16*>(g.C) + m * g.ldc;
  *reinterpret_cast<uint2*>(C + n) = pack4_bf16(gu[0], gu[1], gu[2], gu[3]);
  *reinterpret_cast<uint2*>(C + g.glu_f + n) = pack4_bf16(gv[0], gv[1], gv[2], gv[3]);
}

template <class SH>
__device__ __forceinline__ void glu_bwd_rows(const GemmArgs& g, const float* stage, int r0, int sub, int c, int n,
                                             int M, bool full) {
  const bf16* U = static_cast<const bf16*>(g.aux);
  const int64_t ldu = 2ll * g.glu_f;
  if (full) {
#pragma unroll
    for (int h = 0; h < SH::NIT / 8; ++h) {
      uint2 ur[8], vr[8];
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int64_t m = r0 + SH::RPI * (8 * h + it);
        ur[it] = *reinterpret_cast<const uint2*>(U + m * ldu + n);
        vr[it] = *reinterpret_cast<const uint2*>(U + m * ldu + g.glu_f + n);
      }
#pragma unroll
      for (int it = 0; it < 8; ++it) {
        const int r = SH::RPI * (8 * h + it);
        const float4 gs = *reinterpret_cast<const float4*>(stage + (r + sub) * SH::Pitch + c);
        glu_bwd_one(g, gs, ur[it], vr[it], r0 + r, n);
      }
    }
  } else {
#pragma unroll 1
    for (int it = 0; it < SH::NIT; ++it) {
      const int64_t m = r0 + SH::RPI * it;
      if (m >= M || n >= g.N) continue;
      const float4 gs = *reinterpret_cast<const float4*>(stage + (SH::RPI * it + sub) * SH::Pitch + c);
      glu_bwd_one(g, gs, *reinterpret_cast<const uint2*>(U + m * ldu + n),
                  *reinterpret_cast<const uint2*>(U + m * ldu + g.glu_f + n), m, n);
    }
  }
}

// Fused squared-ReLU forward: staged values (alpha applied) of rows r0 + 2 it,
// columns n..n+3, go to C (if given) as u (bf16, kept for the backward) and to aux as
// s = relu(u)^2 of the float32 u (one rounding fewer than from a stored u).
__device__ __forceinline__ void relu2_fwd_one(const GemmArgs& g, float4 v, int64_t m, int n) {
  const float u[4] = {v.x, v.y, v.z, v.w};
  float q[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float z = fmaxf(u[e], 0.f);
    q[e] = z * z;
  }
  if (g.C) *reinterpret_cast<uint2*>(static_cast<bf16*>(g.C) + m * g.ldc + n) = pack4_bf16(u[0], u[1], u[2], u[3]);
  *reinterpret_cast<uint2*>(static_cast<bf16*>(g.aux) + m * g.glu_f + n) = pack4_bf16(q[0], q[1], q[2], q[3]);
}

template <class SH>
__device__ __forceinline__ void relu2_fwd_rows(const GemmArgs& g, const float* stage, int r0, int sub, int c,
                                               int n, int M, bool full) {
  if (full) {
#pragma unroll
    for (int it = 0; it < SH::NIT; ++it)
      relu2_fwd_one(g, *reinterpret_cast<const float4*>(stage + (SH::RPI * it + sub) * SH::Pitch + c), r0 + SH::RPI * it, n);
  } else {
#pragma unroll 1
    for (int it = 0; it < SH::NIT; ++it) {
      const int64_t m = r0 + SH::RPI * it;
      if (m >= M || n >= g.N) continue;
      relu2_fwd_one(g, *reinterpret_cast<const float4*>(stage + (SH::RPI * it + sub) * SH::Pitch + c), m, n);
    }
  }
}

// Fused squared-ReLU backward: the staged gs values, kept in float32 (gs is
// never stored), with u read from aux, give gu = gs 2 relu(u) in C.
__device__ __forceinline__ void relu2_bwd_one(const GemmArgs& g, float4 gs, uint2 ur, int64_t m, int n) {
  const float4 u = unpack4_bf16(ur);
  *reinterpret_cast<uint2*>(static_cast<bf16*>(g.C) + m * g.ldc + n) =
      pack4_bf16(gs.x * 2.f * fmaxf(u.x, 0.f), gs.y * 2.f * fmaxf(u.y, 0.f), gs.z * 2.f * fmaxf(u.z, 0.f),
                 gs.w * 2.f * fmaxf(u.w, 0.f));
}

template <class SH>
__device__ __forceinline__ void relu2_bwd_rows(const GemmArgs& g, const float* stage, int r0, int sub, int c,
                                               int n, int M, bool full) {
  const bf16* U = static_cast<const bf16*>(g.aux);
  if (full) {
    uint2 ur[SH::NIT];
#pragma unroll
    for (int it = 0; it < SH::NIT; ++it) ur[it] = *reinterpret_cast<const uint2*>(U + static_cast<int64_t>(r0 + SH::RPI * it) * g.glu_f + n);
#pragma unroll
    for (int it = 0; it < SH::NIT; ++it)
      relu2_bwd_one(g, *reinterpret_cast<const float4*>(stage + (SH::RPI * it + sub) * SH::Pitch + c), ur[it],
                    r0 + SH::RPI * it, n);
  } else {
#pragma unroll 1
    for (int it = 0; it < SH::NIT; ++it) {
      const int64_t m = r0 + SH::RPI * it;
      if (m >= M || n >= g.N) continue;
      relu2_bwd_one(g, *reinterpret_cast<const float4*>(stage + (SH::RPI * it + sub) * SH::Pitch + c),
                    *reinterpret_cast<const uint2*>(U + m * g.glu_f + n), m, n);
    }
  }
}

// Plain bf16 output of a 32-row block row that crosses M: straight from the
// accumulators, each row checked (lane: row 16 ii + l16, columns 16 j + q16).
template <int NJ>
__device__ __forceinline__ void epilogue_plain_edge_bf16(const GemmArgs& g, const floatx4 (&a0)[NJ],
                                                         const floatx4 (&a1)[NJ], float alpha, int mb, int nb,
                                                         int l16, int q16, int M) {
#pragma unroll
  for (int ii = 0; ii < 2; ++ii) {
    const int m = mb + 16 * ii + l16;
    if (m < M) {
      bf16* C = static_cast<bf16*>(g.C) + static_cast<int64_t>(m) * g.ldc + nb + q16;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const floatx4& a = ii ? a1[j] : a0[j];
        store_b4(C + j * 16, alpha * a[0], alpha * a[1], alpha * a[2], alpha * a[3]);
      }
    }
  }
}

// One workgroup's tile of a GEMM: `pid` in [0, n_tiles) picks the tile
// (n_tiles covers every row the grid was sized for), `sp` of `splits` the
// k range; `ring` is the workgroup's LDS.
template <bool AK, bool BKC, int EPI = kEpiPlain, int BM = 256>
__device__ __forceinline__ void gemm_big_body(const GemmArgs& g, bf16* ring, int pid, int n_tiles, int sp,
                                              int splits) {
  using SH = BigShape<BM>;
  constexpr int NJ = SH::NJ, WC = SH::WC;
  int M, K;
  resolve_counts(g, M, K);
  const int tiles_n = (g.N + GB - 1) / GB;
  const int tiles_m = min(n_tiles / tiles_n, (M + BM - 1) / BM);
  int tm, tn;
  if (!tile_coords(pid, tiles_m, tiles_n, tm, tn)) return;
  const int m0 = tm * BM, n0 = tn * GB;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / SH::NWN, wn = wave % SH::NWN;
  const bf16* A = static_cast<const bf16*>(g.A);
  const bf16* B = static_cast<const bf16*>(g.B);

  // k range of this split
  const int nkt_all = (K + GK - 1) / GK;
  const int kt0 = static_cast<int>((static_cast<int64_t>(nkt_all) * sp) / splits);
  const int kt1 = static_cast<int>((static_cast<int64_t>(nkt_all) * (sp + 1)) / splits);
  const int nk = kt1 - kt0;
  const int kend = min(K, kt1 * GK);  // loads at or past it read zeros

  floatx4 acc[4][NJ];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v) acc[i][j][v] = 0.f;

  const OpLanes<AK> oa = op_lanes<AK>(g.lda, lane, wave, wm * 64);
  const OpLanes<BKC> ob = op_lanes<BKC>(g.ldb, lane, wave, wn * WC);
  const int64_t ea = mc_extent(kend, M, g.lda), eb = mc_extent(kend, g.N, g.ldb);
  bf16* const ra = ring;                     // A's slots
  bf16* const rb = ring + SH::NSA * SH::SlotA;  // B's slots
  // Load instruction q of A or B for k step kt into slot sl.
  auto load_a = [&](int sl, int kt, int q) {
    tile_part<AK>(ra + sl * SH::SlotA, oa, A, g.lda, ea, m0, M, (kt0 + kt) * GK, kend, wave, q);
  };
  auto load_b = [&](int sl, int kt, int q) {
    if constexpr (EPI == kEpiGluFwd)
      tile_part_glu<WC>(rb + sl * kSlot, ob, B, g.ldb, tn, g.glu_f, (kt0 + kt) * GK, kend, wave, q);
    else
      tile_part<BKC>(rb + sl * kSlot, ob, B, g.ldb, eb, n0, g.N, (kt0 + kt) * GK, kend, wave, q);
  };
  // The compiler's own loads (the kept count among them) are done with here:
  // left pending on some path, it would wait for one -- for every load of
  // the ring -- inside the k loop (11% of the backward pair launches).
  __builtin_amdgcn_s_waitcnt(kWaitVm0);
  if constexpr (BM == 256) {
    // Steps 0 and 1; A's step 2 goes out in step 0's first quarter.
#pragma unroll
    for (int q = 0; q < kLoads; ++q) load_b(0, 0, q);
#pragma unroll
    for (int q = 0; q < kLoads; ++q) load_a(0, 0, q);
#pragma unroll
    for (int q = 0; q < kLoads; ++q) load_a(1, 1, q);
#pragma unroll
    for (int q = 0; q < kLoads; ++q) load_b(1, 1, q);
    dma_barrier<2 * kLoads>();  // step 0 has landed
    bf16x8 fa[2][4], fb[2][4];  // A blocks per k-substep, B blocks per half
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[0][i] = frag<AK>(ra, oa, i, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) fb[0][j] = frag<BKC>(rb, ob, j, 0);
    int sa = 0;  // A's slot of step kt
    for (int kt = 0; kt < nk; ++kt) {
      const int sb = kt & 1;
      const int sa1 = sa == 2 ? 0 : sa + 1, sa2 = sa1 == 2 ? 0 : sa1 + 1;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        const int ks = h >> 1, P = h & 1, nks = ((h + 1) >> 1) & 1;
        const bf16* na = ra + (h == 3 ? sa1 : sa) * kSlot;
        const bf16* nb = rb + (h == 3 ? sb ^ 1 : sb) * kSlot;
        // all of step kt is read; step kt+1 has landed (in flight: A's kt+2)
        if (h == 3) dma_barrier<kLoads>();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int i = q >> 2, j = q & 3;
          acc[i][4 * P + j] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[P][j], fa[ks][i], acc[i][4 * P + j], 0, 0, 0);
          if (P == 0) {  // the other four B blocks
            if (q < 8 && (q & 1) == 0) fb[1][q >> 1] = frag<BKC>(nb, ob, 4 + (q >> 1), ks);
          } else if (q < 8) {  // the next k-substep's A blocks and first B blocks
            if (q & 1)
              fa[ks ^ 1][q >> 1] = frag<AK>(na, oa, q >> 1, nks);
            else
              fb[0][q >> 1] = frag<BKC>(nb, ob, q >> 1, nks);
          }
          if ((q & 3) == 0) {
            if (h == 3) load_b(sb, kt + 2, q >> 2);
            if (h == 0) load_a(sa2, kt + 2, q >> 2);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      sa = sa1;
    }
  } else {
    // Half the rows: two halves of 16 MFMAs per k step, one per k-substep, the
    // barrier before the second.  Three slots of each operand, so step kt+3
    // follows into step kt's slots: B's loads after the barrier, A's in the
    // next step's first half (the first fill leaves step 2's to step 0).
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int q = 0; q < kLoads; ++q) load_b(t, t, q);
#pragma unroll
      for (int q = 0; q < SH::LoadsA; ++q) load_a(t, t, q);
    }
#pragma unroll
    for (int q = 0; q < kLoads; ++q) load_b(2, 2, q);
    dma_barrier<2 * kLoads + SH::LoadsA>();  // step 0 has landed
    bf16x8 fa[2][4], fb[2][4];               // per k-substep
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      fa[0][i] = frag<AK>(ra, oa, i, 0);
      fb[0][i] = frag<BKC>(rb, ob, i, 0);
    }
    int sl = 0;  // slots of step kt
    for (int kt = 0; kt < nk; ++kt) {
      const int sl1 = sl == 2 ? 0 : sl + 1, sl2 = sl1 == 2 ? 0 : sl1 + 1;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bf16* na = ra + (h == 1 ? sl1 : sl) * SH::SlotA;
        const bf16* nb = rb + (h == 1 ? sl1 : sl) * kSlot;
        // all of step kt is read; step kt+1 has landed (in flight: step kt+2)
        if (h == 1) dma_barrier<kLoads + SH::LoadsA>();
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const int i = q >> 2, j = q & 3;
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[h][j], fa[h][i], acc[i][j], 0, 0, 0);
          if (q < 8) {
            if (q & 1)
              fa[h ^ 1][q >> 1] = frag<AK>(na, oa, q >> 1, h ^ 1);
            else
              fb[h ^ 1][q >> 1] = frag<BKC>(nb, ob, q >> 1, h ^ 1);
          }
          if (h == 1 && (q & 3) == 0) load_b(sl, kt + 3, q >> 2);
          if (h == 0 && (q & 7) == 0) load_a(sl2, kt + 2, q >> 3);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      sl = sl1;
    }
  }

  // Epilogue staged through LDS.  A lane holds, per 16x16 block, one output
  // row and 4 consecutive columns; stored directly that scatters every store
  // over 16 rows.  Instead each wave writes one block row of its results
  // (32 x WC float32, alpha applied) into a private [32][Pitch] block
  // and reads it back row-major: WC / 4 lanes then cover WC contiguous
  // columns of one row, so the residual loads and the output stores (one
  // rounding, after the residual) are fully coalesced.  The blocks are
  // private to the wave, so after one barrier (the ring's last loads have
  // landed everywhere) only the wave's own LDS accesses are ordered: no
  // workgroup barrier, whose memory fence would wait for every store in
  // flight, and the stores drain while the wave goes on.
  const float alpha = g.alpha * (g.alpha_dev ? *g.alpha_dev : 1.f);
  const int sub = lane / (WC / 4);
  const int l16 = lane & 15, q16 = 4 * (lane >> 4);
  float* part = g.part ? g.part + static_cast<int64_t>(sp) * g.M * g.N : nullptr;
  float* stage = reinterpret_cast<float*>(ring) + wave * (32 * SH::Pitch);
  const int c = (lane % (WC / 4)) * 4;
  const int n = n0 + wn * WC + c;
  // A block row takes the branch-free path when all its 32 rows and WC
  // columns are in range.
  const bool full_cols = n0 + wn * WC + WC <= g.N;
  // Largest kept sequence index, for the row map (rows < M only).
  const int q_last = g.out_map.idx && M > 0 ? (M - 1) / g.out_map.S : 0;
  dma_barrier<0>();  // the loop's last loads (zeros) land before the ring is reused
  // A plain bf16 output (no residual, row map or partials) is rounded as it
  // is staged: half the LDS traffic, and 16-byte stores that cover a row's
  // 128 columns with 16 lanes (four rows per instruction).  The same single
  // rounding of alpha * acc as the float32 staging gives.  Block rows that
  // cross M store straight from the accumulators, row by row.
  if constexpr (EPI == kEpiGluFwd) {
    // [u v] and s are bf16 outputs too, staged as bf16 the same way; rows
    // past M are not stored
    {
      bf16* st16 = reinterpret_cast<bf16*>(stage);
      constexpr int GW = WC / 2;                                  // the wave's d_ff columns
      constexpr int LU = WC / 8, LS = GW / 8;                     // lanes per row of [u v], of s
      const int rr = lane / LU, cc = (lane % LU) * 8;             // [u v]: the lane's row and columns cc..cc+7
      const int rs = lane / LS, cs = (lane % LS) * 8;             // s
      const int f0 = tn * 128 + wn * GW;                          // the wave's first d_ff column
      bf16* C = static_cast<bf16*>(g.C);
      bf16* Sp = static_cast<bf16*>(g.aux);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int mb = m0 + wm * 64 + i * 32;
        if (mb >= M) break;
        if (C) {  // [u v], unless nothing reads them later
#pragma unroll
          for (int ii = 0; ii < 2; ++ii)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
              const floatx4& a = acc[2 * i + ii][j];
              *reinterpret_cast<uint2*>(st16 + (16 * ii + l16) * SH::Pitch + j * 16 + q16) =
                  pack4_bf16(alpha * a[0], alpha * a[1], alpha * a[2], alpha * a[3]);
            }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          // staged columns below GW are gate (u) columns, the others up (v) columns
          const int gcol = cc < GW ? f0 + cc : g.glu_f + f0 + cc - GW;
#pragma unroll
          for (int k = 0; k < LU / 2; ++k) {
            const int row = 64 / LU * k + rr;
            const bf16* src = st16 + row * SH::Pitch + cc;
            const uint2 lo = *reinterpret_cast<const uint2*>(src), hi = *reinterpret_cast<const uint2*>(src + 4);
            if (mb + row < M)
              *reinterpret_cast<uint4*>(C + static_cast<int64_t>(mb + row) * g.ldc + gcol) =
                  make_uint4(lo.x, lo.y, hi.x, hi.y);
          }
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        }
        // s = silu(u) v from the float32 accumulators (see below)
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
          for (int j = 0; j < NJ / 2; ++j) {
            float sv[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              sv[e] = swiglu_fwd_f(alpha * acc[2 * i + ii][j][e], alpha * acc[2 * i + ii][j + NJ / 2][e]);
            *reinterpret_cast<uint2*>(st16 + (16 * ii + l16) * SH::Pitch + j * 16 + q16) =
                pack4_bf16(sv[0], sv[1], sv[2], sv[3]);
          }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int k = 0; k < LS / 2; ++k) {
          const int row = 64 / LS * k + rs;
          const bf16* src = st16 + row * SH::Pitch + cs;
          const uint2 lo = *reinterpret_cast<const uint2*>(src), hi = *reinterpret_cast<const uint2*>(src + 4);
          if (mb + row < M)
            *reinterpret_cast<uint4*>(Sp + static_cast<int64_t>(mb + row) * g.glu_f + f0 + cs) =
                make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // reads done before the block is rewritten
      }
      return;
    }
  }
  if constexpr (EPI == kEpiPlain || EPI == kEpiKv) {
    if (!part && !g.R && !g.c_f32 && !g.out_map.idx && full_cols) {
      bf16* st16 = reinterpret_cast<bf16*>(stage);
      constexpr int LU = WC / 8;                       // lanes per row
      const int rr = lane / LU, cc = (lane % LU) * 8;  // read: the lane's row and columns cc..cc+7
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int mb = m0 + wm * 64 + i * 32;
        if (mb + 32 > M) {
          if (mb < M) epilogue_plain_edge_bf16(g, acc[2 * i], acc[2 * i + 1], alpha, mb, n0 + wn * WC, l16, q16, M);
          continue;
        }
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            const floatx4& a = acc[2 * i + ii][j];
            *reinterpret_cast<uint2*>(st16 + (16 * ii + l16) * SH::Pitch + j * 16 + q16) =
                pack4_bf16(alpha * a[0], alpha * a[1], alpha * a[2], alpha * a[3]);
          }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // rows are 2 WC + 8 bytes apart (8-byte aligned, no bank conflicts for the
        // 8-byte stage writes), so each 16 bytes are read as two 8-byte halves
        uint4 v[LU / 2];
#pragma unroll
        for (int k = 0; k < LU / 2; ++k) {
          const bf16* src = st16 + (64 / LU * k + rr) * SH::Pitch + cc;
          const uint2 lo = *reinterpret_cast<const uint2*>(src), hi = *reinterpret_cast<const uint2*>(src + 4);
          v[k] = make_uint4(lo.x, lo.y, hi.x, hi.y);
        }
        bf16* C = static_cast<bf16*>(g.C);
#pragma unroll
        for (int k = 0; k < LU / 2; ++k)
          store_b8(C + static_cast<int64_t>(mb + 64 / LU * k + rr) * g.ldc + n0 + wn * WC + cc, v[k]);
        if constexpr (EPI == kEpiKv) {
          // the key and value columns once more, into the cache; S % 32 == 0,
          // so the block row lies in one sequence
          const int col = n0 + wn * WC + cc - g.kv_d, b = mb / g.kv_S;
          if (col >= 0) {
            bf16* kv = static_cast<bf16*>(g.kv) + (static_cast<int64_t>(b) * g.kv_s_max + mb - b * g.kv_S) * 2 * g.kv_d + col;
#pragma unroll
            for (int k = 0; k < LU / 2; ++k)
              *reinterpret_cast<uint4*>(kv + static_cast<int64_t>(64 / LU * k + rr) * 2 * g.kv_d) = v[k];
          }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // reads done before the block is rewritten
      }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const floatx4& a = acc[2 * i + ii][j];
        *reinterpret_cast<float4*>(stage + (16 * ii + l16) * SH::Pitch + j * 16 + q16) =
            make_float4(alpha * a[0], alpha * a[1], alpha * a[2], alpha * a[3]);
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // staged values visible to the wave
    const int mb = m0 + wm * 64 + i * 32;              // first row of the block row
    if constexpr (EPI == kEpiGluBwd) {
      glu_bwd_rows<SH>(g, stage, mb + sub, sub, c, n, M, n0 + wn * WC + WC <= g.N && mb + 32 <= M);
    } else if constexpr (EPI == kEpiRelu2Fwd) {
      relu2_fwd_rows<SH>(g, stage, mb + sub, sub, c, n, M, n0 + wn * WC + WC <= g.N && mb + 32 <= M);
    } else if constexpr (EPI == kEpiRelu2Bwd) {
      relu2_bwd_rows<SH>(g, stage, mb + sub, sub, c, n, M, n0 + wn * WC + WC <= g.N && mb + 32 <= M);
    } else {
      if (full_cols && mb + 32 <= M)
        epilogue_rows_full<SH>(g, part, stage, mb + sub, sub, c, n, q_last);
      else
        epilogue_rows_edge<SH>(g, part, stage, mb + sub, sub, c, n, M);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // reads done before the block is rewritten
  }
}

#define LD_BIG_ATTRS __global__ __launch_bounds__(kBigThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
#define LD_BIG_KERNEL(name, ak, bk)                                                    \
  LD_BIG_ATTRS void name(GemmArgs g) {                                                 \
    __shared__ __align__(16) bf16 ring[kRingElems];                          \
    gemm_big_body<ak, bk>(g, ring, blockIdx.x, gridDim.x, blockIdx.y, gridDim.y);      \
  }
LD_BIG_KERNEL(ld_gemm_bf16_nt_256, true, true)
LD_BIG_KERNEL(ld_gemm_bf16_nn_256, true, false)
LD_BIG_KERNEL(ld_gemm_bf16_tn_256, false, false)
LD_BIG_KERNEL(ld_gemm_bf16_tt_256, false, true)

// C = [u v] rows and aux = silu(u) v rows of the SwiGLU projection (see GemmArgs).
LD_BIG_ATTRS void ld_gemm_bf16_nt_glu_256(GemmArgs g) {
  __shared__ __align__(16) bf16 ring[kRingElems];
  gemm_big_body<true, true, kEpiGluFwd>(g, ring, blockIdx.x, gridDim.x, 0, 1);
}

// C = u rows and aux = relu(u)^2 rows of the squared-ReLU projection (see GemmArgs).
LD_BIG_ATTRS void ld_gemm_bf16_nt_relu2_256(GemmArgs g) {
  __shared__ __align__(16) bf16 ring[kRingElems];
  gemm_big_body<true, true, kEpiRelu2Fwd>(g, ring, blockIdx.x, gridDim.x, 0, 1);
}

// The forward projections on 128-row tiles (see plan_rows).
LD_BIG_ATTRS void ld_gemm_bf16_nt_128(GemmArgs g) {
  __shared__ __align__(16) bf16 ring[kRingElems];
  gemm_big_body<true, true, kEpiPlain, 128>(g, ring, blockIdx.x, gridDim.x, 0, 1);
}
LD_BIG_ATTRS void ld_gemm_bf16_nt_glu_128(GemmArgs g) {
  __shared__ __align__(16) bf16 ring[kRingElems];
  gemm_big_body<true, true, kEpiGluFwd, 128>(g, ring, blockIdx.x, gridDim.x, 0, 1);
}
LD_BIG_ATTRS void ld_gemm_bf16_nt_relu2_128(GemmArgs g) {
  __shared__ __align__(16) bf16 ring[kRingElems];
  gemm_big_body<true, true, kEpiRelu2Fwd, 128>(g, ring, blockIdx.x, gridDim.x, 0, 1);
}

// The QKV projection of an evaluation with a cache: key and value columns also
// go there (see GemmArgs).  3264 x 6144 x 2048: 89.9 -> 90.4 us, in place of a
// launch of 9.7 us that read them back; a kernel of its own, so the other plain
// GEMMs' registers and code stay as they are.
LD_BIG_ATTRS void ld_gemm_bf16_nt_kv_256(GemmArgs g) {
  __shared__ __align__(16) bf16 ring[kRingElems];
  gemm_big_body<true, true, kEpiKv>(g, ring, blockIdx.x, gridDim.x, 0, 1);
}
LD_BIG_ATTRS void ld_gemm_bf16_nt_kv_128(GemmArgs g) {
  __shared__ __align__(16) bf16 ring[kRingElems];
  gemm_big_body<true, true, kEpiKv, 128>(g, ring, blockIdx.x, gridDim.x, 0, 1);
}

// Up to three GEMMs in one launch: weight-gradient GEMMs g1 (tiles1 tiles,
// each split into splits1 k ranges) and g3 (tiles3 tiles, never split; both
// with both operands mn-contiguous) and an input-gradient GEMM g2 (A
// k-contiguous, B mn-contiguous, tiles2 tiles).  The workgroups go in the
// order g3, g1, g2, or g2 first (g2_first); the later GEMMs' workgroups
// fill the CUs the earlier ones leave idle, so no GEMM's last partial round
// runs on a part-empty chip.  tiles1 = tiles3 = 0 leaves g2 alone.
template <int EPI2>
__device__ __forceinline__ void gemm_pair_body(const GemmArgs& g1, const GemmArgs& g3, const GemmArgs& g2, int tiles1,
                                               int splits1, int tiles3, int tiles2, int g2_first) {
  __shared__ __align__(16) bf16 ring[kRingElems];
  const int n1 = tiles1 * splits1;
  int id = blockIdx.x;
  if (g2_first) {
    if (id < tiles2) {
      gemm_big_body<true, false, EPI2>(g2, ring, id, tiles2, 0, 1);
      return;
    }
    id -= tiles2;
  } else if (id >= tiles3 + n1) {
    gemm_big_body<true, false, EPI2>(g2, ring, id - tiles3 - n1, tiles2, 0, 1);
    return;
  }
  if (id < tiles3)
    gemm_big_body<false, false>(g3, ring, id, tiles3, 0, 1);
  else
    gemm_big_body<false, false>(g1, ring, (id - tiles3) % tiles1, tiles1, (id - tiles3) / tiles1, splits1);
}
LD_BIG_ATTRS void ld_gemm_bf16_tn_nn_256(GemmArgs g1, GemmArgs g3, GemmArgs g2, int tiles1, int splits1, int tiles3,
                                         int tiles2, int g2_first) {
  gemm_pair_body<kEpiPlain>(g1, g3, g2, tiles1, splits1, tiles3, tiles2, g2_first);
}
// The same with the SwiGLU backward fused into g2's epilogue (see GemmArgs).
LD_BIG_ATTRS void ld_gemm_bf16_tn_nn_glu_256(GemmArgs g1, GemmArgs g3, GemmArgs g2, int tiles1, int splits1,
                                             int tiles3, int tiles2, int g2_first) {
  gemm_pair_body<kEpiGluBwd>(g1, g3, g2, tiles1, splits1, tiles3, tiles2, g2_first);
}
// The same with the squared-ReLU backward fused into g2's epilogue.
LD_BIG_ATTRS void ld_gemm_bf16_tn_nn_relu2_256(GemmArgs g1, GemmArgs g3, GemmArgs g2, int tiles1, int splits1,
                                               int tiles3, int tiles2, int g2_first) {
  gemm_pair_body<kEpiRelu2Bwd>(g1, g3, g2, tiles1, splits1, tiles3, tiles2, g2_first);
}

// C[i] = sum over splits of part[s][i], float32, in split order.  Every
// split's value is requested before the first add (splits <= kMaxSplits).
constexpr int kMaxSplits = 8;
__global__ __launch_bounds__(256) void ld_splitk_reduce(const float* part, int splits, int64_t mn, float* C) {
  for (int64_t i4 = blockIdx.x * 256ll + threadIdx.x; i4 < mn / 4; i4 += gridDim.x * 256ll) {
    float4 t[kMaxSplits];
#pragma unroll
    for (int k = 0; k < kMaxSplits; ++k)
      if (k < splits) t[k] = reinterpret_cast<const float4*>(part + static_cast<int64_t>(k) * mn)[i4];
    float4 sum = t[0];
#pragma unroll
    for (int k = 1; k < kMaxSplits; ++k)
      if (k < splits) {
        sum.x += t[k].x; sum.y += t[k].y; sum.z += t[k].z; sum.w += t[k].w;
      }
    store_f4(C + 4 * i4, sum);
  }
}

// Dynamic LDS limit of the 128x128 kernels, raised once per process (a
// function-local static: its initialisation is thread-safe).
void set_attrs() {
  static const bool done = [] {
    const void* small[] = {reinterpret_cast<const void*>(ld_gemm_bf16_nt),
                           reinterpret_cast<const void*>(ld_gemm_bf16_nn),
                           reinterpret_cast<const void*>(ld_gemm_bf16_tn),
                           reinterpret_cast<const void*>(ld_gemm_bf16_tt)};
    for (const void* f : small) (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kGemmLds);
    return true;
  }();
  (void)done;
}

}  // namespace

constexpr int kCus = 256;   // compute units the plans are made for
constexpr int kPlanK = 32;  // unit of k in the launch estimates

static int64_t big_tiles_of(int64_t M, int64_t N, int bm) { return ((M + bm - 1) / bm) * ((N + GB - 1) / GB); }

static int64_t f32_tiles(const GemmArgs& g, int64_t max_m) { return ((max_m + 63) / 64) * ((g.N + 63) / 64); }

// Whether a float32 GEMM takes ld_gemm_f32_vec_k: 16-byte aligned rows whose ends
// the 4-wide loads meet exactly.  At K <= 16 half of its k tile is padding and
// there is no next one to load ahead: with tiles for every CU the plain kernel
// takes less (16384 x 2048 x 16 66 -> 53 us; 16384 x 64 x 16, B not k-contiguous,
// 13.4 -> 9.2; both operands mn-contiguous, where its loads are the slower ones,
// from 1024 tiles up).
static bool f32_vec(int a_kcontig, int b_kcontig, const GemmArgs& g, int64_t max_m) {
  const bool vec = reinterpret_cast<uintptr_t>(g.A) % 16 == 0 && reinterpret_cast<uintptr_t>(g.B) % 16 == 0 &&
                   g.lda % 4 == 0 && g.ldb % 4 == 0 && ((!a_kcontig && !b_kcontig) || g.K % 4 == 0) &&
                   (a_kcontig || g.M % 4 == 0) && (b_kcontig || g.N % 4 == 0);
  const bool shallow = g.K <= FK && !(g.dev_count && g.count_dim) &&
                       f32_tiles(g, max_m) >= (a_kcontig || b_kcontig ? kCus : 1024);
  return vec && !shallow;
}

// The 128x128 kernel of a layout.
const char* gemm_kernel_name(int a_kcontig, int b_kcontig) {
  if (a_kcontig) return b_kcontig ? "ld_gemm_bf16_nt" : "ld_gemm_bf16_nn";
  return b_kcontig ? "ld_gemm_bf16_tt" : "ld_gemm_bf16_tn";
}

// A last round of tiles that leaves most of the 256 CUs idle costs as much as a
// full one; 128-row tiles halve what a round costs, at 0.56-0.6 of a 256-row
// tile's time each (8192 x 8192 x 8192 1.15 times as long, a third more
// operand traffic per product).  So they are taken where the rounds, weighted
// with that, are fewer: 3264 x 2048 x 5504 (104 or 208 tiles) 95 -> 66 us,
// 3264 x 6144 x 2048 (312 or 624) 88 -> 82, 8192 x 768 x 2048 (96 or 192) 41 -> 27;
// 8192 x 4096 x 768 (512 or 1024) stays at 50 (59).
constexpr double kHalfTile = 0.59;

int plan_rows(int64_t m, int64_t n) {
  auto rounds = [&](int bm) { return static_cast<double>((big_tiles_of(m, n, bm) + kCus - 1) / kCus); };
  return kHalfTile * rounds(128) < rounds(256) ? 128 : 256;
}

GemmPlan plan_gemm(int dtype, int a_kcontig, int b_kcontig, const GemmArgs& g, int64_t max_m,
                   int64_t max_k, bool allow_split, int64_t host_m) {
  GemmPlan p{};
  p.splits = 1;
  p.bm = GB;
  if (dtype != LD_BF16) {
    p.name = f32_vec(a_kcontig, b_kcontig, g, max_m) ? "ld_gemm_f32_vec_k" : "ld_gemm_f32_k";
    return p;
  }
  const int64_t big_tiles = ((max_m + GB - 1) / GB) * ((g.N + GB - 1) / GB);
  // the big tile's epilogue stores 4 consecutive columns at once
  // each operand is addressed through one buffer descriptor: spans < 2 GiB (an
  // mn-contiguous one is fetched 64 k rows at a time, whatever K is, with
  // 32-bit offsets that must not wrap back into it)
  const int64_t k_rows = std::max<int64_t>(max_k, GK);
  const int64_t a_span = 2 * g.lda * (a_kcontig ? max_m : k_rows);
  const int64_t b_span = 2 * g.ldb * (b_kcontig ? static_cast<int64_t>(g.N) : k_rows);
  // split-K only for float32 outputs without a residual (weight gradients);
  // such a GEMM fills the CUs through its splits even with few tiles
  const bool splittable = allow_split && g.c_f32 && !g.R && !g.out_map.idx && g.ldc == g.N && max_k >= 16 * kPlanK;
  // The big kernel takes every size (at 64 rows of 2048 columns and K = 2048,
  // a few tiles, the 128x128 one takes 33 us and it 23; NN 60 and 41): the
  // 128x128 kernel is for operands its 16-byte loads into LDS do not take and
  // widths its stores of 4 columns do not.
  auto aligned = [](const void* q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; };
  p.big = g.N % 4 == 0 && g.ldc % 4 == 0 && (!g.R || g.ldr % 4 == 0) && aligned(g.A) && aligned(g.B) &&
          a_span < kBigMaxSpan && b_span < kBigMaxSpan;
  if (p.big) {
    if (splittable) {
      double best = 0;
      for (int s = 1; s <= kMaxSplits; ++s) {
        const int64_t wg = big_tiles * s;
        const double eff = static_cast<double>(wg) / (1.0 * kCus * ((wg + kCus - 1) / kCus)) - 0.02 * (s - 1);
        if (eff > best + 1e-9 && max_k / s >= 8 * kPlanK) {
          best = eff;
          p.splits = s;
        }
      }
    }
    if (a_kcontig && b_kcontig && p.splits == 1) p.bm = plan_rows(host_m > 0 ? host_m : max_m, g.N);
    p.name = a_kcontig && b_kcontig ? (p.bm == 128 ? "ld_gemm_bf16_nt_128" : "ld_gemm_bf16_nt_256")
             : a_kcontig            ? "ld_gemm_bf16_nn_256"
             : b_kcontig            ? "ld_gemm_bf16_tt_256"
                                    : "ld_gemm_bf16_tn_256";
  } else {
    p.name = gemm_kernel_name(a_kcontig, b_kcontig);
  }
  return p;
}

// Where a GEMM on its own takes less on the 128x128 kernel than on the ring one:
// a few k steps over a ragged edge.  The ring kernel's edge block rows are
// stored row by row, and their code and its first fills cost about 2 us more than
// the small kernel's, which a few k steps do not make up.  us on 128x128 and ring:
//   B or A mn-contiguous, columns no multiple of 128, at most a tile per CU (two of
//   at most 32 columns): NN 2048 x 264 x 64 10.2 and 12.1, x 128 11.6 and 13.0, x 256
//   15.4 and 15.7, 8192 x 776 x 128 (448 tiles) 15.9 and 14.0; TN 2048 x 136 x 64 10.3
//   and 10.9, x 128 12.0 and 11.5; NN 2048 x 32 x 256 12.3 and 15.4, x 512 18.9 and
//   19.7, 65536 x 32 x 64 9.0 and 12.8.
//   Both k-contiguous, at most 96 columns, no multiple of a wave's, too many rows
//   for one round of 128-row ring tiles: 65536 x 32 x 64 8.2 and 12.2, x 64 x 512 20.2
//   and 21.7, x 96 x 192 15.2 and 15.8, x 96 x 512 22.7 and 22.3; but 66000 x 64 x 64,
//   on 128-row tiles without an edge, 17.7 and 13.6.
bool gemm_prefers_small(const GemmPlan& p, int a_kcontig, int b_kcontig, const GemmArgs& g, int64_t max_m) {
  if (!p.big || p.splits > 1 || g.kv || (g.dev_count && g.count_dim)) return false;
  if (a_kcontig && b_kcontig)
    return g.N <= 96 && g.N % (p.bm == 128 ? 64 : 128) != 0 && big_tiles_of(max_m, g.N, 128) > kCus &&
           g.K <= (g.N <= 64 ? 1024 : 192);
  const int64_t tiles = ((max_m + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  const int most_k = g.N <= 32 ? (a_kcontig || b_kcontig ? 384 : 128) : a_kcontig || b_kcontig ? 128 : 64;
  return g.N % BN != 0 && tiles <= (g.N <= 32 ? 2 * kCus : kCus) && g.K <= most_k;
}

// Whole block rows and columns only (an edge is stored on another path), and
// 16-byte pieces that stay within the key and value columns.
bool gemm_stores_kv(const GemmPlan& p, const GemmArgs& g) {
  return p.big && !g.R && !g.c_f32 && !g.dev_count && !g.out_map.idx && g.N % GB == 0 && g.kv_d % 8 == 0 &&
         g.N == 3 * g.kv_d && g.kv_S % 32 == 0 && g.M % 32 == 0 && reinterpret_cast<uintptr_t>(g.kv) % 16 == 0;
}

size_t gemm_part_bytes(const GemmPlan& p, int64_t M, int64_t N) {
  return p.splits > 1 ? 4ull * p.splits * M * N : 0;
}

hipError_t launch_gemm_plan(int dtype, int a_kcontig, int b_kcontig, const GemmPlan& p, GemmArgs g,
                            int64_t max_m, hipStream_t s) {
  if (max_m <= 0 || g.N <= 0) return hipSuccess;
  if (dtype == LD_BF16 && p.big) {
    set_attrs();
    const int64_t tiles = big_tiles_of(max_m, g.N, p.bm);
    float* C = static_cast<float*>(g.C);
    if (p.splits > 1) {
      if (!g.part) return hipErrorInvalidValue;
    } else {
      g.part = nullptr;
    }
    const dim3 grid(static_cast<unsigned>(tiles), p.splits), block(kBigThreads);
    if (g.kv) {
      if (p.splits != 1 || !gemm_stores_kv(p, g)) return hipErrorInvalidValue;
      if (p.bm == 128)
        hipLaunchKernelGGL(ld_gemm_bf16_nt_kv_128, grid, block, 0, s, g);
      else
        hipLaunchKernelGGL(ld_gemm_bf16_nt_kv_256, grid, block, 0, s, g);
    } else if (a_kcontig && b_kcontig && p.bm == 128)
      hipLaunchKernelGGL(ld_gemm_bf16_nt_128, grid, block, 0, s, g);
    else if (a_kcontig && b_kcontig)
      hipLaunchKernelGGL(ld_gemm_bf16_nt_256, grid, block, 0, s, g);
    else if (a_kcontig)
      hipLaunchKernelGGL(ld_gemm_bf16_nn_256, grid, block, 0, s, g);
    else if (b_kcontig)
      hipLaunchKernelGGL(ld_gemm_bf16_tt_256, grid, block, 0, s, g);
    else
      hipLaunchKernelGGL(ld_gemm_bf16_tn_256, grid, block, 0, s, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.splits == 1) return e;
    const int64_t mn = static_cast<int64_t>(g.M) * g.N;
    int blocks = static_cast<int>(std::min<int64_t>((mn / 4 + 255) / 256, 1 << 20));
    hipLaunchKernelGGL(ld_splitk_reduce, dim3(blocks), dim3(256), 0, s, g.part, p.splits, mn, C);
    return hipGetLastError();
  }
  return launch_gemm(dtype, a_kcontig, b_kcontig, g, max_m, s);
}

// Estimated finish time, in k tiles of 32, of classes of workgroups (count, cost
// each) dealt in launch order to n_cu CUs, one workgroup per CU, each CU taking
// the next when it frees.
static double list_schedule(std::initializer_list<std::pair<int64_t, double>> classes, int n_cu) {
  std::priority_queue<double, std::vector<double>, std::greater<double>> cu;
  for (int i = 0; i < n_cu; ++i) cu.push(0.0);
  double end = 0.0;
  for (const auto& c : classes)
    for (int64_t w = 0; w < c.first; ++w) {
      const double t = cu.top() + c.second;
      cu.pop();
      cu.push(t);
      end = std::max(end, t);
    }
  return end;
}

PairPlan plan_gemm_pair(int64_t m1, int64_t n1, int64_t k1, int64_t m3, int64_t n3, int64_t m2, int64_t n2,
                        int64_t k2, int max_splits) {
  struct Entry {
    int64_t key[9];
    PairPlan plan;
  };
  constexpr int kEntries = 64;  // the kept counts of a step give a few dozen shapes
  thread_local Entry cache[kEntries];
  thread_local int next = 0;
  const int64_t key[9] = {m1, n1, k1, m3, n3, m2, n2, k2, max_splits};
  for (const Entry& e : cache)
    if (std::equal(key, key + 9, e.key)) return e.plan;
  // Fitted to the four-wave kernel with k tiles of 32 that the ring kernel replaced
  // (which takes about 0.78 us per 32 k); only their ratios weigh in the choice.
  constexpr double kEpi = 8.0;       // epilogue of one tile, in k-tile times
  constexpr double kLaunch = 4.0;    // a second (reduction) launch
  constexpr double kTileUs = 0.95;   // one k tile of 32 on one CU
  auto tiles = [](int64_t m, int64_t n) { return ((m + GB - 1) / GB) * ((n + GB - 1) / GB); };
  const int64_t tiles1 = m1 > 0 ? tiles(m1, n1) : 0, tiles3 = m3 > 0 ? tiles(m3, n3) : 0;
  const int64_t tiles2 = tiles(m2, n2);
  const int64_t nkt1 = (k1 + kPlanK - 1) / kPlanK;
  const double c2 = static_cast<double>((k2 + kPlanK - 1) / kPlanK) + kEpi;
  const double c3 = static_cast<double>(nkt1) + kEpi;
  PairPlan best{1, 0, 0.0};
  double best_t = 0.0;
  for (int sp = 1; sp <= (tiles1 > 0 ? max_splits : 1); ++sp) {
    const double c1 = static_cast<double>((nkt1 + sp - 1) / sp) + kEpi;
    for (int order = 0; order < 2; ++order) {
      double t = order ? list_schedule({{tiles2, c2}, {tiles3, c3}, {tiles1 * sp, c1}}, kCus)
                       : list_schedule({{tiles3, c3}, {tiles1 * sp, c1}, {tiles2, c2}}, kCus);
      if (sp > 1)  // partials written and read back at ~5 TB/s, plus a launch
        t += kLaunch + (sp + 1.0) * 4.0 * m1 * n1 / 5e12 / (kTileUs * 1e-6);
      if ((sp == 1 && order == 0) || t < best_t - 1e-9) {
        best_t = t;
        best = PairPlan{sp, order, t};
      }
    }
  }
  Entry& e = cache[next];
  next = (next + 1) % kEntries;
  std::copy(key, key + 9, e.key);
  e.plan = best;
  return best;
}

hipError_t launch_gemm_glu_fwd(const GemmArgs& g, int64_t max_m, int bm, hipStream_t s) {
  if (max_m <= 0 || g.N <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(big_tiles_of(max_m, g.N, bm))), block(kBigThreads);
  if (bm == 128)
    hipLaunchKernelGGL(ld_gemm_bf16_nt_glu_128, grid, block, 0, s, g);
  else
    hipLaunchKernelGGL(ld_gemm_bf16_nt_glu_256, grid, block, 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gemm_relu2_fwd(const GemmArgs& g, int64_t max_m, int bm, hipStream_t s) {
  if (max_m <= 0 || g.N <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(big_tiles_of(max_m, g.N, bm))), block(kBigThreads);
  if (bm == 128)
    hipLaunchKernelGGL(ld_gemm_bf16_nt_relu2_128, grid, block, 0, s, g);
  else
    hipLaunchKernelGGL(ld_gemm_bf16_nt_relu2_256, grid, block, 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gemm_pair(GemmArgs g1, const GemmArgs* g3, const PairPlan& p, const GemmArgs& g2, int64_t max_m2,
                            hipStream_t s) {
  const int splits1 = p.splits1;
  const int64_t tiles1 =
      g1.M > 0 ? ((static_cast<int64_t>(g1.M) + GB - 1) / GB) * ((g1.N + GB - 1) / GB) : 0;
  const int64_t tiles3 =
      g3 ? ((static_cast<int64_t>(g3->M) + GB - 1) / GB) * ((g3->N + GB - 1) / GB) : 0;
  const int64_t tiles2 = ((max_m2 + GB - 1) / GB) * ((g2.N + GB - 1) / GB);
  if (splits1 > 1) {
    if (!g1.part) return hipErrorInvalidValue;
  } else {
    g1.part = nullptr;
  }
  const GemmArgs g3v = g3 ? *g3 : g1;
  const int64_t wg = tiles1 * splits1 + tiles3 + tiles2;
  if (wg <= 0) return hipSuccess;
  if (g2.relu2)
    hipLaunchKernelGGL(ld_gemm_bf16_tn_nn_relu2_256, dim3(static_cast<unsigned>(wg)), dim3(kBigThreads), 0, s, g1, g3v, g2,
                       static_cast<int>(tiles1), splits1, static_cast<int>(tiles3), static_cast<int>(tiles2),
                       p.g2_first);
  else if (g2.glu_f > 0)
    hipLaunchKernelGGL(ld_gemm_bf16_tn_nn_glu_256, dim3(static_cast<unsigned>(wg)), dim3(kBigThreads), 0, s, g1, g3v, g2,
                       static_cast<int>(tiles1), splits1, static_cast<int>(tiles3), static_cast<int>(tiles2),
                       p.g2_first);
  else
    hipLaunchKernelGGL(ld_gemm_bf16_tn_nn_256, dim3(static_cast<unsigned>(wg)), dim3(kBigThreads), 0, s, g1, g3v, g2,
                       static_cast<int>(tiles1), splits1, static_cast<int>(tiles3), static_cast<int>(tiles2),
                       p.g2_first);
  return hipGetLastError();
}

hipError_t launch_splitk_reduce(const float* part, int splits, int64_t mn, float* C, hipStream_t s) {
  if (splits <= 1 || mn <= 0) return hipSuccess;
  const int blocks = static_cast<int>(std::min<int64_t>((mn / 4 + 255) / 256, 1 << 20));
  hipLaunchKernelGGL(ld_splitk_reduce, dim3(blocks), dim3(256), 0, s, part, splits, mn, C);
  return hipGetLastError();
}

template <int TS>
static hipError_t launch_f32_vec(int a_kcontig, int b_kcontig, const GemmArgs& g, int64_t max_m, hipStream_t s) {
  const int64_t tiles = ((max_m + TS - 1) / TS) * ((g.N + TS - 1) / TS);
  const dim3 grid(static_cast<unsigned>(tiles)), block(256);
  if (a_kcontig && b_kcontig)
    hipLaunchKernelGGL((ld_gemm_f32_vec_k<true, true, TS>), grid, block, 0, s, g);
  else if (a_kcontig)
    hipLaunchKernelGGL((ld_gemm_f32_vec_k<true, false, TS>), grid, block, 0, s, g);
  else if (b_kcontig)
    hipLaunchKernelGGL((ld_gemm_f32_vec_k<false, true, TS>), grid, block, 0, s, g);
  else
    hipLaunchKernelGGL((ld_gemm_f32_vec_k<false, false, TS>), grid, block, 0, s, g);
  return hipGetLastError();
}

hipError_t launch_gemm(int dtype, int a_kcontig, int b_kcontig, const GemmArgs& g, int64_t max_m, hipStream_t s) {
  if (max_m <= 0 || g.N <= 0) return hipSuccess;
  if (dtype == LD_BF16) {
    set_attrs();
    const int64_t tiles = ((max_m + BM - 1) / BM) * ((g.N + BN - 1) / BN);
    const dim3 grid(static_cast<unsigned>(tiles)), block(256);
    if (a_kcontig && b_kcontig)
      hipLaunchKernelGGL(ld_gemm_bf16_nt, grid, block, kGemmLds, s, g);
    else if (a_kcontig)
      hipLaunchKernelGGL(ld_gemm_bf16_nn, grid, block, kGemmLds, s, g);
    else if (b_kcontig)
      hipLaunchKernelGGL(ld_gemm_bf16_tt, grid, block, kGemmLds, s, g);
    else
      hipLaunchKernelGGL(ld_gemm_bf16_tn, grid, block, kGemmLds, s, g);
    return hipGetLastError();
  }
  if (f32_vec(a_kcontig, b_kcontig, g, max_m)) {
    // 64 x 64 tiles do twice the arithmetic per LDS read; below a tile per CU
    // the latency of a tile counts, and 32 x 32 ones spread it over more CUs
    return f32_tiles(g, max_m) >= kCus ? launch_f32_vec<64>(a_kcontig, b_kcontig, g, max_m, s)
                                       : launch_f32_vec<32>(a_kcontig, b_kcontig, g, max_m, s);
  }
  const int64_t tiles = ((max_m + FT - 1) / FT) * ((g.N + FT - 1) / FT);
  const dim3 grid(static_cast<unsigned>(tiles)), block(256);
  if (a_kcontig && b_kcontig)
    hipLaunchKernelGGL((ld_gemm_f32_k<true, true>), grid, block, 0, s, g);
  else if (a_kcontig)
    hipLaunchKernelGGL((ld_gemm_f32_k<true, false>), grid, block, 0, s, g);
  else if (b_kcontig)
    hipLaunchKernelGGL((ld_gemm_f32_k<false, true>), grid, block, 0, s, g);
  else
    hipLaunchKernelGGL((ld_gemm_f32_k<false, false>), grid, block, 0, s, g);
  return hipGetLastError();
}

}  // namespace ld
