// The end of a loss call: loss partials -> statistics, by one block.
#pragma once
#include "mrl_internal.h"

namespace mrl {

constexpr int EPI_NQ = 10;   // doubles per block in loss_partials
// loss_partials layout per block: 0 pg, 1 kl, 2 sgt, 3 sum_ratio, 4 max_ratio, 5 sum_k3,
// 6 n_clipped, 7 n_zero_grad, 8 n_grpo_tokens, 9 n_saturated_rows

__device__ inline double wave_sum64(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}
__device__ inline double wave_max64(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { const double o = __shfl_xor(x, off); x = o > x ? o : x; }
  return x;
}

// All threads of a block of THREADS call it.  (Partials are added per thread in order, then by wave: the same sums from run to
// run.)
template <int THREADS>
__device__ inline void finalize_block(const FinalizeArgs& a) {
  // rows the enqueued passes did not cover (only when the caller's hint was too small)
  for (int64_t i = a.rows_enqueued + threadIdx.x; i < *a.n_scored; i += THREADS)
    a.out_logp[a.row_index[i]] = __builtin_nanf("");
  __shared__ double sh[THREADS / 64][EPI_NQ];
  __shared__ double tot[EPI_NQ];
  double q[EPI_NQ];
#pragma unroll
  for (int k = 0; k < EPI_NQ; ++k) q[k] = 0.0;
  for (int64_t b = threadIdx.x; b < a.n_blocks; b += THREADS) {
#pragma unroll
    for (int k = 0; k < EPI_NQ; ++k) {
      const double v = a.parts[b * EPI_NQ + k];
      q[k] = k == 4 ? (v > q[k] ? v : q[k]) : q[k] + v;
    }
  }
#pragma unroll
  for (int k = 0; k < EPI_NQ; ++k) {
    const double v = k == 4 ? wave_max64(q[k]) : wave_sum64(q[k]);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < EPI_NQ) {
    double acc = 0.0;
    for (int w = 0; w < THREADS / 64; ++w) {
      const double v = sh[w][threadIdx.x];
      acc = threadIdx.x == 4 ? (v > acc ? v : acc) : acc + v;
    }
    tot[threadIdx.x] = acc;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const double ng = tot[8];
    a.out_d[0] = tot[0] + (double)a.beta * tot[1] + (double)a.lambda * tot[2];
    a.out_d[1] = tot[0];
    a.out_d[2] = tot[1];
    a.out_d[3] = tot[2];
    a.out_d[4] = ng > 0 ? tot[3] / ng : 0.0;
    a.out_d[5] = tot[4];
    a.out_d[6] = ng > 0 ? tot[5] / ng : 0.0;
    a.out_i[0] = *a.n_scored;
    a.out_i[1] = (int64_t)(tot[6] + 0.5);
    a.out_i[2] = (int64_t)(tot[7] + 0.5);
    a.out_i[3] = *a.n_bad;
    a.out_i[4] = *a.n_scored > a.rows_enqueued ? *a.n_scored - a.rows_enqueued : 0;
    a.out_i[5] = (int64_t)(tot[9] + 0.5);
  }
}

}  // namespace mrl
