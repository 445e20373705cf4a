// fp32 GEMM C[m][n] = sum_k A[m][k] * B[n][k] of the small-shape path (dtype MRL_F32), on the fp32 MFMA
// (v_mfma_f32_16x16x4_f32: fp32 products and sums).
//
// The shapes are a few hundred rows and columns, so a launch is a handful of tiles and what it takes is
// latency: the four waves of a block split the contraction (every fourth 16-wide step each) and add their
// accumulators through LDS in wave order; operands go from global memory (the L2, at these sizes) straight
// into the registers of the MFMA, four k values per lane and load, several steps in flight.  A lane's four
// k values feed four MFMAs, element e of lane group q being k = 4 q + e for A and B alike, so a step is
// 16 wide and needs no LDS.  Operands may be k-contiguous or k-major (rows of the source are k), so that
// nothing is transposed in memory.
// Tile 16 x 16 per block; 32 x 32 from kBigTiles tiles on, where the chip is full and halving the operand
// reads counts for more.  256 slots, V = 512, d = 64, against a 64 x 64 tile per block through LDS and
// transposed operands: forward 12.3 -> 3.4 us, dH 77 (+ 4.8 for the transpose) -> 6.7 us, dW 38 (+ 4.7) -> 4.7 us.
#include "mrl_finalize.h"
#include "mrl_internal.h"

namespace mrl {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kStep = 16;
constexpr int64_t kBigTiles = 512;

// Four values k .. k + 3 of operand row `row` (already mapped and in range), zero from K on.  The loads
// are unconditional (clamped indices, selected values), so that several steps' loads can be in
// flight.  A k-contiguous operand is read with one 16-byte load that needs 4-byte alignment only;
// TAIL: K is no multiple of 4, and the last load of a row, moved back into it, is shifted (odd widths
// read value by value run at half the rate: 4096 x 515 x 10001 1675 us against 758 us).
enum { LOAD_EXACT, LOAD_TAIL, LOAD_SINGLE };
template <bool KMAJOR, int LOAD>
__device__ inline f32x4 load4(const float* p, int64_t ld, const int32_t* k_rows, int64_t row, int k, int K) {
  f32x4 v;
  if (KMAJOR || LOAD == LOAD_SINGLE) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int kk = k + e < K ? k + e : K - 1;
      const float x = KMAJOR ? p[(k_rows ? (int64_t)k_rows[kk] : (int64_t)kk) * ld + row] : p[row * ld + kk];
      v[e] = k + e < K ? x : 0.f;
    }
  } else {
    const int kk = k + 4 <= K ? k : K - 4;
    const f32x4 u = *reinterpret_cast<const f32x4_any*>(p + row * ld + kk);
    const int back = k - kk;                          // > 0: the wanted values start at u[back]
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = u[e];
      if (LOAD == LOAD_TAIL) {
        x = back == 1 ? (e < 3 ? u[e < 3 ? e + 1 : 3] : 0.f) : x;
        x = back == 2 ? (e < 2 ? u[e < 2 ? e + 2 : 3] : 0.f) : x;
        x = back == 3 ? (e < 1 ? u[3] : 0.f) : x;
        x = back >= 4 ? 0.f : x;
      } else {
        x = back > 0 ? 0.f : x;
      }
      v[e] = x;
    }
  }
  return v;
}

template <int N> struct Const { static constexpr int value = N; };

template <int T> using Parts = f32x4[4][T * T][64];   // the waves' accumulators

// tile (mb, nb) of one product
template <int T, bool A_KMAJOR, bool B_KMAJOR>
__device__ inline void tile_f32(const GemmF32Args& a, int mb, int nb, Parts<T>& part) {
  int M = a.M, K = a.K;
  if (a.m_dynamic || a.k_dynamic) {
    int64_t r = *a.n_scored - a.chunk_start;
    const int nv = r < 0 ? 0 : (r > a.chunk_rows ? a.chunk_rows : (int)r);
    if (a.m_dynamic) M = nv;
    if (a.k_dynamic) K = nv;
  }
  const int m0 = mb * (16 * T), n0 = nb * (16 * T);
  if (m0 >= M) return;
  if (a.k_dynamic && K == 0 && a.accumulate) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, q = lane >> 4;
  int64_t arow[T], brow[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int m = m0 + 16 * t + r < M ? m0 + 16 * t + r : M - 1;
    arow[t] = !A_KMAJOR && a.a_rows ? (int64_t)a.a_rows[m] : (int64_t)m;
    brow[t] = n0 + 16 * t + r < a.N ? n0 + 16 * t + r : a.N - 1;
  }
  f32x4 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto contract = [&](auto load) {
    constexpr int LOAD = decltype(load)::value;
    for (int k0 = wave * kStep; k0 < K; k0 += 4 * kStep) {
      f32x4 av[T], bv[T];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        av[t] = load4<A_KMAJOR, LOAD>(a.A, a.lda, a.a_rows, arow[t], k0 + 4 * q, K);
        bv[t] = load4<B_KMAJOR, LOAD>(a.B, a.ldb, a.b_rows, brow[t], k0 + 4 * q, K);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][e], bv[j][e], acc[i][j], 0, 0, 0);
    }
  };
  if (K % 4 == 0) contract(Const<LOAD_EXACT>{});
  else if (K > 4) contract(Const<LOAD_TAIL>{});
  else contract(Const<LOAD_SINGLE>{});
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) part[wave][i * T + j][lane] = acc[i][j];
  __syncthreads();
  // one output per thread and 16 x 16 sub-tile; lane 16 q + c of an accumulator holds rows 4 q .. 4 q + 3 of column c
  const int mm = threadIdx.x >> 4, c = threadIdx.x & 15;
  const int src = (mm >> 2) * 16 + c, e = mm & 3;
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) {
      const int m = m0 + 16 * i + mm, n = n0 + 16 * j + c;
      if (m >= M || n >= a.N) continue;
      const int s = i * T + j;
      const float v = (part[0][s][src][e] + part[1][s][src][e]) + (part[2][s][src][e] + part[3][s][src][e]);
      const int64_t crow = a.c_rows ? (int64_t)a.c_rows[m] : (int64_t)m;
      float* dst = a.C + crow * a.ldc + n;
      if (a.accumulate) *dst += v; else *dst = v;
    }
}

template <int T, bool A_KMAJOR, bool B_KMAJOR>
__global__ __launch_bounds__(256) void k_gemm_f32(GemmF32Args a) {
  __shared__ Parts<T> part;
  tile_f32<T, A_KMAJOR, B_KMAJOR>(a, a.m_on_x ? blockIdx.x : blockIdx.y, a.m_on_x ? blockIdx.y : blockIdx.x, part);
}

// dH and dW of a small pass in one launch: both read dz and neither fills the chip (a call of 256 slots,
// V = 512, d = 64, which the host bounds: 39.9 -> 33.7 - 35.7 us).  Blocks below
// `first` are tiles of a, in rows of a_cols, the others up to `tiles` tiles of b, in rows of b_cols; a block behind them,
// if there is one, ends the call (256 slots, V = 512, d = 64: with a launch of its own 28.6 us a call, now 23.8).
__global__ __launch_bounds__(256) void k_gemm_f32_pair(GemmF32Args a, int a_cols, int first, GemmF32Args b, int b_cols, int tiles,
                                                       FinalizeArgs last) {
  __shared__ Parts<1> part;
  const int t = blockIdx.x;
  if (t == tiles) { finalize_block<256>(last); return; }
  if (t < first) tile_f32<1, false, true>(a, t / a_cols, t % a_cols, part);
  else tile_f32<1, true, true>(b, (t - first) / b_cols, (t - first) % b_cols, part);
}

bool is_big(const GemmF32Args& a) { return (int64_t)((a.N + 31) / 32) * ((a.M + 31) / 32) >= kBigTiles; }

template <bool A_KMAJOR, bool B_KMAJOR>
void launch(GemmF32Args a, hipStream_t stream) {
  const bool big = is_big(a);
  const int tile = big ? 32 : 16;
  const unsigned mt = (a.M + tile - 1) / tile, nt = (a.N + tile - 1) / tile;
  a.m_on_x = mt > nt;                                 // the longer side: y is limited to 65535
  const dim3 grid(a.m_on_x ? mt : nt, a.m_on_x ? nt : mt);
  if (big) hipLaunchKernelGGL((k_gemm_f32<2, A_KMAJOR, B_KMAJOR>), grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL((k_gemm_f32<1, A_KMAJOR, B_KMAJOR>), grid, dim3(256), 0, stream, a);
}

}  // namespace

bool gemm_f32_pairs(const GemmF32Args& a, const GemmF32Args& b) { return !is_big(a) && !is_big(b); }

void launch_gemm_f32_pair(const GemmF32Args& a, const GemmF32Args& b, const FinalizeArgs* last, hipStream_t stream) {
  const int a_cols = (a.N + 15) / 16, b_cols = (b.N + 15) / 16;
  const int first = a_cols * ((a.M + 15) / 16), blocks = first + b_cols * ((b.M + 15) / 16);
  hipLaunchKernelGGL(k_gemm_f32_pair, dim3(blocks + (last != nullptr ? 1 : 0)), dim3(256), 0, stream, a, a_cols, first, b, b_cols,
                     blocks, last != nullptr ? *last : FinalizeArgs{});
}

void launch_gemm_f32(const GemmF32Args& a, hipStream_t stream) {
  if (a.a_kmajor) launch<true, true>(a, stream);
  else if (a.b_kmajor) launch<false, true>(a, stream);
  else launch<false, false>(a, stream);
}

}  // namespace mrl
