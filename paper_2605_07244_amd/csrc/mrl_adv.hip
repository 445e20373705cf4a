// Group-relative advantages (Sec. 3), pool-wide (Sec. 5.1) and pooled-baseline
// (App. I.1) variants, and the SGT gate flags (Sec. 5.3 / App. B).
//
// One wavefront per group finds its members among all B entries (B is a few thousand:
// the whole input is a few KB and stays in L2), so group members need not be contiguous
// and every sum has a fixed order: lane-strided partial sums in fp64, then a
// fixed butterfly.  Mean and variance are taken in two passes so that binary
// rewards give exact zeros for all-equal groups.
#include "mrl_internal.h"

namespace mrl {
namespace {

__device__ inline double wave_sum(double x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}
__device__ inline int wave_sum_i(int x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

struct AdvArgs {
  const float* rewards; const int32_t* group_id;
  const uint8_t* in_stats; const uint8_t* scored; const uint8_t* is_own; const float* baseline_shift;
  int64_t B; int G; int mode; float eps_norm; int ddof; float mix_alpha;
  float neg_thresh, pos_thresh;
  float* out_adv; float* out_mean; float* out_std; uint8_t* out_flags;
};

// The entries of the wave's group among b = lane, lane + 64, ...: up to 64 steps of the wave are
// remembered as a bit mask, so that a batch of up to kRemembered entries is scanned once (all group
// ids loaded independently of each other) and the three passes touch the group's own entries only;
// larger batches are scanned in every pass, kScanSteps ids at a time.  1024 entries, 128 groups: 1.5 + 9.6 us in
// two launches, 5.7 us now; a call of 20000 entries, 5 groups 295 us before this structure, 302 with one id at a
// time, 237 with four, 8192 entries, 1024 groups 57, 56 and 34.
constexpr int64_t kRemembered = 64 * 64;
constexpr int kScanSteps = 4;
struct Members {
  const int32_t* group_id; int64_t B; int g; uint64_t bits; bool remembered;
  __device__ Members(const int32_t* ids, int64_t n, int group, int lane) : group_id(ids), B(n), g(group), bits(0), remembered(n <= kRemembered) {
    if (!remembered) return;
    const int n32 = (int)n;
    for (int s0 = 0; s0 * 64 < n32; s0 += 16) {
      int id[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int b = (s0 + k) * 64 + lane;
        id[k] = b < n32 ? ids[b] : -1;
      }
#pragma unroll
      for (int k = 0; k < 16; ++k) bits |= (uint64_t)(id[k] == group) << ((s0 + k) & 63);
    }
  }
  template <class F> __device__ void each(int lane, F f) const {   // in ascending order
    if (remembered) {
      for (uint64_t m = bits; m != 0; m &= m - 1) f((int64_t)__builtin_ctzll(m) * 64 + lane);
    } else {
      for (int64_t b0 = lane; b0 < B; b0 += 64 * kScanSteps) {
        int id[kScanSteps];
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) id[k] = b0 + 64 * k < B ? group_id[b0 + 64 * k] : -1;
#pragma unroll
        for (int k = 0; k < kScanSteps; ++k) if (id[k] == g) f(b0 + 64 * k);
      }
    }
  }
};

// Blocks below group_blocks: one wave per group.  The blocks behind them clear the entries whose group
// id is outside [0, G), which no wave owns.
__global__ __launch_bounds__(256) void k_group_adv(AdvArgs a, int group_blocks) {
  if ((int)blockIdx.x >= group_blocks) {
    const int64_t b = (int64_t)(blockIdx.x - group_blocks) * 256 + threadIdx.x;
    if (b < a.B && (a.group_id[b] < 0 || a.group_id[b] >= a.G)) a.out_adv[b] = 0.f;
    return;
  }
  const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (g >= a.G) return;
  const int lane = threadIdx.x & 63;
  const Members members(a.group_id, a.B, g, lane);
  // pass 1: counts, sums, gate predicates
  double sum_p = 0.0, sum_o = 0.0;
  int cnt_p = 0, cnt_o = 0, n_own = 0, own_not_fail = 0, peer_succ = 0;
  members.each(lane, [&](int64_t b) {
    const float r = a.rewards[b];
    const bool st = a.in_stats == nullptr || a.in_stats[b] != 0;
    const bool own = a.is_own == nullptr || a.is_own[b] != 0;
    if (st) { sum_p += (double)r; cnt_p++; if (own) { sum_o += (double)r; cnt_o++; } }
    // (no if / else over the two counters: by reference it becomes one counter behind a selected address,
    // that is, in scratch memory: 326 instead of 302 us for that call)
    n_own += own;
    own_not_fail += own && !(r < a.neg_thresh);
    peer_succ += !own && r > a.pos_thresh;
  });
  sum_p = wave_sum(sum_p); sum_o = wave_sum(sum_o);
  cnt_p = wave_sum_i(cnt_p); cnt_o = wave_sum_i(cnt_o);
  n_own = wave_sum_i(n_own); own_not_fail = wave_sum_i(own_not_fail); peer_succ = wave_sum_i(peer_succ);
  const double mu_p = cnt_p > 0 ? sum_p / cnt_p : 0.0;
  const double mu_o = cnt_o > 0 ? sum_o / cnt_o : 0.0;
  // pass 2: squared deviations
  double sq_p = 0.0, sq_o = 0.0;
  members.each(lane, [&](int64_t b) {
    const bool st = a.in_stats == nullptr || a.in_stats[b] != 0;
    if (!st) return;
    const bool own = a.is_own == nullptr || a.is_own[b] != 0;
    const double r = (double)a.rewards[b];
    sq_p += (r - mu_p) * (r - mu_p);
    if (own) sq_o += (r - mu_o) * (r - mu_o);
  });
  sq_p = wave_sum(sq_p); sq_o = wave_sum(sq_o);
  const double sd_p = cnt_p - a.ddof > 0 ? sqrt(sq_p / (cnt_p - a.ddof)) : 0.0;
  const double sd_o = cnt_o - a.ddof > 0 ? sqrt(sq_o / (cnt_o - a.ddof)) : 0.0;
  // pass 3: advantages
  const bool zn = a.mode == 1;
  const double eps = (double)a.eps_norm, alpha = (double)a.mix_alpha;
  // perturbed-baseline control (App. C.4): the shift moves the baseline, not the std
  const double shift = a.baseline_shift != nullptr ? (double)a.baseline_shift[g] : 0.0;
  const double bl_p = mu_p + shift, bl_o = mu_o + shift;
  members.each(lane, [&](int64_t b) {
    const bool sc = a.scored == nullptr || a.scored[b] != 0;
    double adv = 0.0;
    if (sc) {
      const double r = (double)a.rewards[b];
      const double ap = cnt_p > 0 ? (zn ? (r - bl_p) / (sd_p + eps) : r - bl_p) : 0.0;
      if (a.mix_alpha == 1.0f) {
        adv = ap;
      } else {
        const double ao = cnt_o > 0 ? (zn ? (r - bl_o) / (sd_o + eps) : r - bl_o) : 0.0;
        adv = (1.0 - alpha) * ao + alpha * ap;
      }
    }
    a.out_adv[b] = (float)adv;
  });
  if (lane == 0) {
    if (a.out_mean) a.out_mean[g] = (float)mu_p;
    if (a.out_std) a.out_std[g] = (float)sd_p;
    if (a.out_flags) {
      const bool all_fail = n_own > 0 && own_not_fail == 0;
      const bool ps = peer_succ > 0;
      a.out_flags[g] = (uint8_t)((all_fail ? 1u : 0u) | (ps ? 2u : 0u) | ((all_fail && ps) ? 4u : 0u));
    }
  }
}

// batch normalisation (App. A): divide the group-centred advantages of scored,
// in-range entries by their std over the batch (+ eps); single block, fixed order.
__global__ __launch_bounds__(1024) void k_adv_batch_scale(const int32_t* group_id, const uint8_t* scored,
                                                         int64_t B, int G, float eps_norm, int ddof,
                                                         float* adv) {
  __shared__ double sh[16];
  __shared__ int shc[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double s = 0.0;
  int c = 0;
  for (int64_t b = threadIdx.x; b < B; b += 1024) {
    const bool sc = (scored == nullptr || scored[b] != 0) && group_id[b] >= 0 && group_id[b] < G;
    if (sc) { s += (double)adv[b]; c++; }
  }
  s = wave_sum(s);
  c = wave_sum_i(c);                                  // (B is at most 2^30)
  if (lane == 0) { sh[wave] = s; shc[wave] = c; }
  __syncthreads();
  double total = 0.0;
  int cnt = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) { total += sh[w]; cnt += shc[w]; }
  const double mu = cnt > 0 ? total / (double)cnt : 0.0;
  double q = 0.0;
  for (int64_t b = threadIdx.x; b < B; b += 1024) {
    const bool sc = (scored == nullptr || scored[b] != 0) && group_id[b] >= 0 && group_id[b] < G;
    if (sc) { const double dlt = (double)adv[b] - mu; q += dlt * dlt; }
  }
  q = wave_sum(q);
  __syncthreads();
  if (lane == 0) sh[wave] = q;
  __syncthreads();
  double sq = 0.0;
#pragma unroll
  for (int w = 0; w < 16; ++w) sq += sh[w];
  const double sd_s = cnt - ddof > 0 ? sqrt(sq / (double)(cnt - ddof)) : 0.0;
  const double denom = sd_s + (double)eps_norm;
  for (int64_t b = threadIdx.x; b < B; b += 1024) {
    const bool sc = (scored == nullptr || scored[b] != 0) && group_id[b] >= 0 && group_id[b] < G;
    if (sc) adv[b] = (float)((double)adv[b] / denom);
  }
}

}  // namespace

void launch_group_advantages(const float* rewards, const int32_t* group_id, const uint8_t* in_stats,
                             const uint8_t* scored, const uint8_t* is_own, const float* baseline_shift,
                             int64_t B, int G, int mode, float eps_norm, int ddof, float mix_alpha, float neg_thresh,
                             float pos_thresh, float* out_adv, float* out_mean, float* out_std,
                             uint8_t* out_flags, hipStream_t stream) {
  AdvArgs a = {rewards, group_id, in_stats, scored, is_own, baseline_shift, B, G, mode, eps_norm, ddof, mix_alpha,
               neg_thresh, pos_thresh, out_adv, out_mean, out_std, out_flags};
  const int group_blocks = (G + 3) / 4;
  hipLaunchKernelGGL(k_group_adv, dim3((unsigned)(group_blocks + (B + 255) / 256)), dim3(256), 0, stream, a, group_blocks);
  if (mode == 2)
    hipLaunchKernelGGL(k_adv_batch_scale, dim3(1), dim3(1024), 0, stream, group_id, scored, B, G, eps_norm,
                       ddof, out_adv);
}

}  // namespace mrl
