// THL word-level trace alignment on integer word maps (Sec. 4.3; App. D, Alg. 2):
// the source model's log-probs are summed per textual word and each word total is
// spread evenly over the target tokens of that word.  One workgroup per sequence;
// per-word sums and counts live in LDS.  The sums are accumulated as 64-bit fixed
// point (2^-32 units) with integer LDS atomics, so the result does not depend on
// the order in which tokens arrive: runs are bit-reproducible.
#include "../../include/mrl.h"
#include "mrl_internal.h"

namespace mrl {
namespace {

constexpr int THL_THREADS = 256;
constexpr int THL_MAX_WORDS = 8192;                 // 8 B sum + 4 B count per word: 96 KB of LDS
constexpr double THL_SCALE = 4294967296.0;          // 2^32

// What bounds the kernel is instruction issue (1180 + 1536 positions a row, a few dozen instructions
// each) on top of a chain of latencies: mask -> rank of the position -> map entry -> per-word sum ->
// output.  Each wave owns a contiguous run of positions, so that a position's rank is the count before
// the wave's run (one exchange through LDS per segment of THL_SEGMENT positions) plus a running
// scalar and a bit count of the mask ballot; the mask bits stay in a register, one per step.  With
// ranks exchanged by two barriers per 256 positions in each of three sweeps, fp64 conversions to
// 64-bit integers and fp64 divisions, 2048 rows (50 MB) took 18.4 us in the kernel and 20.8 a call, now 16.3 and 17.1.
constexpr int THL_WAVES = THL_THREADS / 64;
constexpr int THL_SEGMENT = 32 * THL_THREADS;
constexpr int THL_INVERSES = 64;
constexpr int THL_KEPT = 8;                         // KEEP: steps of a wave at most, rows of 2048 positions
// ... and more than three steps, below which most of what it unrolls is idle.  Calls, us, without and with: 10000 rows of 800 positions
// (four steps) 49.4 and 42.5, of 1024 50.8 and 43.9, 2048 rows 13.2 and 13.4, 14.1 and 13.8; three steps: 10000 rows of
// 600 42.7 and 40.1, but 5000 of 500 + 700 21.5 and 22.6, 2048 of 520 11.7 and 12.4, of 768 12.6 and 12.7; two: 10000
// of 300 + 300 30.2 and 37.8.
constexpr int THL_KEPT_FROM = 3 * THL_THREADS;
constexpr int THL_GROUP = 2;                        // steps whose loads are in flight together (the call: 17.1 us; 4 and 8: 17.7, 1: 18.9)

// round(x * 2^32) to nearest even for |x| < 2^30, with fp32 operations that are all exact but the last
// rounding (scaling by powers of two, integer and fractional parts)
__device__ inline long long to_fixed(float x) {
  const float whole = truncf(x);
  const float f = (x - whole) * 65536.f;             // |f| < 2^16
  const float hi = truncf(f);
  const int lo = (int)rintf((f - hi) * 65536.f);      // |lo| <= 2^16
  return ((long long)(int)whole << 32) + ((long long)(int)hi << 16) + lo;
}

// One side's response tokens within a segment: steps of 64 consecutive positions per wave.  Positions are
// unsigned: rows may have up to 2^31 - 1 of them, and the run of the last segment reaches up to a
// segment beyond.
struct Run {
  uint32_t first; int steps;                                   // first position of the wave's run, its steps
  uint32_t bits;                                      // bit k: this lane's position of step k is a response token
  template <int GROUP = THL_GROUP>
  __device__ void load(const uint8_t* mask, uint32_t j0, uint32_t S, int* wave_counts) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int len = S <= j0 ? 0 : (S - j0 < THL_SEGMENT ? (int)(S - j0) : THL_SEGMENT);
    steps = (len + THL_THREADS - 1) / THL_THREADS;
    first = j0 + wave * steps * 64;
    bits = 0;
    int count = 0;
    for (int k0 = 0; k0 < steps; k0 += GROUP) {
      uint8_t m[GROUP];
#pragma unroll
      for (int k = 0; k < GROUP; ++k) {
        const uint32_t j = first + (k0 + k) * 64 + lane;
        m[k] = mask[j < S ? j : S - 1];
      }
#pragma unroll
      for (int k = 0; k < GROUP; ++k) {
        const bool bit = k0 + k < steps && first + (k0 + k) * 64 + lane < S && m[k] == 1;
        bits |= (uint32_t)bit << ((k0 + k) & 31);
        count += __popcll(__ballot(bit));
      }
    }
    if (lane == 0) wave_counts[wave] = count;
  }
  // tokens before this wave's run (wave_counts published); `total` gets the segment's count
  __device__ int before(const int* wave_counts, int& total) const {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int n = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < THL_WAVES; ++w) { n += w < wave ? wave_counts[w] : 0; total += wave_counts[w]; }
    return n;
  }
  // For the run's positions, THL_GROUP steps at a time: `fetch(k, position, rank)` for the response
  // tokens whose rank is below `limit` (k = step within the group), then `use(k, position, fetched)`
  // for every position of the run, so that the fetches of a group are independent of each other.
  template <class Fetch, class Use> __device__ void each(int rank, int limit, Fetch fetch, Use use) const {
    const int lane = threadIdx.x & 63;
    for (int k0 = 0; k0 < steps; k0 += THL_GROUP) {
      bool in[THL_GROUP];
#pragma unroll
      for (int k = 0; k < THL_GROUP; ++k) {
        const bool bit = k0 + k < steps && ((bits >> ((k0 + k) & 31)) & 1);
        const unsigned long long ball = __ballot(bit);
        const int p = rank + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(ball >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ball, 0u));
        in[k] = bit && p < limit;
        if (in[k]) fetch(k, first + (k0 + k) * 64 + lane, p);
        rank += __popcll(ball);
      }
#pragma unroll
      for (int k = 0; k < THL_GROUP; ++k)
        if (k0 + k < steps) use(k, first + (k0 + k) * 64 + lane, in[k]);
    }
  }
};

// KEEP: rows of more than THL_KEPT_FROM and at most THL_KEPT * THL_THREADS positions.  Their steps are unrolled, masks eight and maps four in flight together,
// and a target token's word stays in a register from the count to the output (32 registers, still eight waves per
// SIMD): 2048 rows of 1180 + 1536 positions 17.1 us a call without, 15.7 with the words kept, 14.7 with both.
template <bool KEEP>
__global__ __launch_bounds__(THL_THREADS) void k_thl_word_align(
    const float* src_logp, const uint8_t* src_mask, const int32_t* src_map, const int32_t* src_map_len,
    const uint8_t* tgt_mask, const int32_t* tgt_map, const int32_t* tgt_map_len, int S_src, int S_tgt,
    int max_words, float ignore_value, float* out, unsigned long long* bad_words) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  long long* wsum = reinterpret_cast<long long*>(smem);                       // [max_words]
  int* wcnt = reinterpret_cast<int*>(smem + (size_t)max_words * 8);           // [max_words]
  __shared__ int counts_s[THL_WAVES], counts_t[THL_WAVES];
  __shared__ double inverse[THL_INVERSES];            // 2^-32 / c
  __shared__ int any_word;
  __shared__ int n_bad;

  const int64_t i = blockIdx.x;
  const float* lp = src_logp + i * S_src;
  const uint8_t* sm = src_mask + i * S_src;
  const int32_t* smap = src_map + i * S_src;
  const uint8_t* tm = tgt_mask + i * S_tgt;
  const int32_t* tmap = tgt_map + i * S_tgt;
  float* o = out + i * S_tgt;
  const int slen = src_map_len[i], tlen = tgt_map_len[i];

  for (int w = threadIdx.x; w < max_words; w += THL_THREADS) { wsum[w] = 0; wcnt[w] = 0; }
  if (threadIdx.x == 0) { any_word = 0; n_bad = 0; }
  if (threadIdx.x < THL_INVERSES) inverse[threadIdx.x] = 1.0 / (THL_SCALE * (double)(threadIdx.x > 0 ? threadIdx.x : 1));

  // aggregation: Z_w = sum of the source log-probs of the response tokens mapped to w, C_w = number of
  // target response tokens mapped to w
  int base_s = 0, base_t = 0, bad_s = 0, bad_t = 0;
  const uint32_t longest = S_src > S_tgt ? S_src : S_tgt;
  Run rs, rt;
  int32_t kept[KEEP ? THL_KEPT : 1];                  // KEEP: the words of this thread's target positions, -1 = none
  for (uint32_t j0 = 0; j0 < longest; j0 += THL_SEGMENT) {
    if (j0 > 0) __syncthreads();                      // the counts of the segment before are consumed
    rs.load<KEEP ? 8 : THL_GROUP>(sm, j0, S_src, counts_s);
    rt.load<KEEP ? 8 : THL_GROUP>(tm, j0, S_tgt, counts_t);
    __syncthreads();                                  // counts; the first time also the cleared words
    int total_s, total_t;
    const int before_s = base_s + rs.before(counts_s, total_s), before_t = base_t + rt.before(counts_t, total_t);
    base_s += total_s;
    base_t += total_t;
    int32_t w[THL_GROUP];
    float x[THL_GROUP];
    if (KEEP) {
      int rank = before_s;
#pragma unroll
      for (int k0 = 0; k0 < THL_KEPT; k0 += 4) {
        int32_t ws[4];
        float xs[4];
        bool in[4];
        if (k0 < rs.steps) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const bool bit = (rs.bits >> (k0 + k)) & 1;
            const unsigned long long ball = __ballot(bit);
            const int p = rank + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(ball >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ball, 0u));
            in[k] = bit && p < slen;
            if (in[k]) { ws[k] = smap[p]; xs[k] = lp[rs.first + (k0 + k) * 64 + (threadIdx.x & 63)]; }
            rank += __popcll(ball);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            if (!in[k]) continue;
            if (ws[k] >= 0 && ws[k] < max_words) {
              atomicAdd(reinterpret_cast<unsigned long long*>(&wsum[ws[k]]), (unsigned long long)to_fixed(xs[k]));
              any_word = 1;
            } else if (ws[k] != -1) {
              ++bad_s;
            }
          }
        }
      }
    } else {
      rs.each(before_s, slen, [&](int k, uint32_t j, int p) { w[k] = smap[p]; x[k] = lp[j]; },
              [&](int k, uint32_t, bool in) {
        if (!in) return;
        if (w[k] >= 0 && w[k] < max_words) {
          atomicAdd(reinterpret_cast<unsigned long long*>(&wsum[w[k]]), (unsigned long long)to_fixed(x[k]));
          any_word = 1;
        } else if (w[k] != -1) {
          ++bad_s;
        }
      });
    }
    if (KEEP) {
      int rank = before_t;
#pragma unroll
      for (int k0 = 0; k0 < THL_KEPT; k0 += 4) {
#pragma unroll
        for (int k = k0; k < k0 + 4; ++k) {
          const bool bit = (rt.bits >> k) & 1;
          const unsigned long long ball = __ballot(bit);
          const int p = rank + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(ball >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ball, 0u));
          kept[k] = -1;
          if (bit && p < tlen) kept[k] = tmap[p];
          rank += __popcll(ball);
        }
#pragma unroll
        for (int k = k0; k < k0 + 4; ++k) {
          if (kept[k] >= 0 && kept[k] < max_words) atomicAdd(&wcnt[kept[k]], 1);
          else { bad_t += kept[k] != -1; kept[k] = -1; }
        }
      }
    } else {
      rt.each(before_t, tlen, [&](int k, uint32_t, int p) { w[k] = tmap[p]; }, [&](int k, uint32_t, bool in) {
        if (!in) return;
        if (w[k] >= 0 && w[k] < max_words) atomicAdd(&wcnt[w[k]], 1);
        else if (w[k] != -1) ++bad_t;
      });
    }
  }
  __syncthreads();
  const bool active = any_word != 0;   // a sequence whose source side carries no word stays inactive

  // redistribution: each target token of word w receives Z_w / C_w.  (An fp64 division is some thirty
  // instructions; the product with the inverse of a small count is within 2^-52 of it before the
  // rounding to fp32.)
  if (KEEP) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < THL_KEPT; ++k) {
      const uint32_t j = rt.first + k * 64 + lane;
      if (k >= rt.steps || j >= (uint32_t)S_tgt) continue;
      float v = ignore_value;
      if (active && kept[k] >= 0) {
        const int c = wcnt[kept[k]];
        v = (float)((double)wsum[kept[k]] * (c < THL_INVERSES ? inverse[c] : 1.0 / (THL_SCALE * (double)c)));
      }
      o[j] = v;
    }
  }
  base_t = 0;
  for (uint32_t j0 = 0; !KEEP && j0 < (uint32_t)S_tgt; j0 += THL_SEGMENT) {
    if (longest > (uint32_t)THL_SEGMENT) {                      // (else the only segment's bits and counts are still there)
      __syncthreads();
      rt.load(tm, j0, S_tgt, counts_t);
      __syncthreads();
    }
    int total_t;
    const int before_t = base_t + rt.before(counts_t, total_t);
    base_t += total_t;
    int32_t w[THL_GROUP];
    rt.each(before_t, tlen, [&](int k, uint32_t, int p) { w[k] = tmap[p]; }, [&](int k, uint32_t j, bool in) {
      if (j >= (uint32_t)S_tgt) return;
      float v = ignore_value;
      if (active && in && w[k] >= 0 && w[k] < max_words) {
        const int c = wcnt[w[k]];
        v = (float)((double)wsum[w[k]] * (c < THL_INVERSES ? inverse[c] : 1.0 / (THL_SCALE * (double)c)));
      }
      o[j] = v;
    });
  }
  if (bad_words != nullptr) {
    const int my_bad = bad_s + (active ? bad_t : 0);
    if (my_bad) atomicAdd(&n_bad, my_bad);
    __syncthreads();
    if (threadIdx.x == 0 && n_bad) atomicAdd(bad_words, (unsigned long long)n_bad);
  }
}

// Rows of at most THL_THREADS positions on either side: one position per thread, in as many waves as the longer
// side (or the clearing of the words) needs, and a target token's word stays in its register from the
// count to the output.  The machinery of the general kernel (runs of steps, groups of two of them, a table of
// inverses) is work without a use here.  A call of 10000 rows of 100 + 100 positions took 17.2 us before that
// kernel, 23.3 with it, 12.5 with this one; 20000 of 64 + 64 25.5, 40.6 and 13.4; 10000 of 250 + 250 22.4, 25.6 and
// 14.2; from two positions per thread on the general one is ahead of the earlier form (300 + 300 34.4 and 29.9).
__global__ __launch_bounds__(THL_THREADS) void k_thl_word_align_short(
    const float* src_logp, const uint8_t* src_mask, const int32_t* src_map, const int32_t* src_map_len,
    const uint8_t* tgt_mask, const int32_t* tgt_map, const int32_t* tgt_map_len, int S_src, int S_tgt,
    int max_words, float ignore_value, float* out, unsigned long long* bad_words) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  long long* wsum = reinterpret_cast<long long*>(smem);                       // [max_words]
  int* wcnt = reinterpret_cast<int*>(smem + (size_t)max_words * 8);           // [max_words]
  __shared__ int counts_s[THL_WAVES], counts_t[THL_WAVES];
  __shared__ int any_word;
  __shared__ int n_bad;

  const int64_t i = blockIdx.x;
  const int j = threadIdx.x, lane = j & 63, wave = __builtin_amdgcn_readfirstlane(j >> 6);
  const uint8_t ms = src_mask[i * S_src + (j < S_src ? j : S_src - 1)], mt = tgt_mask[i * S_tgt + (j < S_tgt ? j : S_tgt - 1)];
  const int slen = src_map_len[i], tlen = tgt_map_len[i];
  const float x = src_logp[i * S_src + (j < S_src ? j : S_src - 1)];
  for (int w = j; w < max_words; w += blockDim.x) { wsum[w] = 0; wcnt[w] = 0; }
  if (j < THL_WAVES) { counts_s[j] = 0; counts_t[j] = 0; }
  if (j == 0) { any_word = 0; n_bad = 0; }
  __syncthreads();
  const bool s = j < S_src && ms == 1, t = j < S_tgt && mt == 1;
  const unsigned long long ball_s = __ballot(s), ball_t = __ballot(t);
  if (lane == 0) { counts_s[wave] = __popcll(ball_s); counts_t[wave] = __popcll(ball_t); }
  __syncthreads();
  int ps = __builtin_amdgcn_mbcnt_hi((uint32_t)(ball_s >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ball_s, 0u));
  int pt = __builtin_amdgcn_mbcnt_hi((uint32_t)(ball_t >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ball_t, 0u));
#pragma unroll
  for (int w = 0; w < THL_WAVES; ++w) { ps += w < wave ? counts_s[w] : 0; pt += w < wave ? counts_t[w] : 0; }
  const bool in_s = s && ps < slen, in_t = t && pt < tlen;
  const int ws = in_s ? src_map[i * S_src + ps] : -1, wt = in_t ? tgt_map[i * S_tgt + pt] : -1;
  const bool word_s = ws >= 0 && ws < max_words, word_t = wt >= 0 && wt < max_words;
  if (word_s) {
    atomicAdd(reinterpret_cast<unsigned long long*>(&wsum[ws]), (unsigned long long)to_fixed(x));
    any_word = 1;
  }
  if (word_t) atomicAdd(&wcnt[wt], 1);
  __syncthreads();
  const bool active = any_word != 0;   // a sequence whose source side carries no word stays inactive
  if (j < S_tgt) out[i * S_tgt + j] = active && word_t ? (float)((double)wsum[wt] / (THL_SCALE * (double)wcnt[wt])) : ignore_value;
  if (bad_words != nullptr) {
    const int my_bad = (!word_s && ws != -1) + (active && !word_t && wt != -1);
    if (my_bad) atomicAdd(&n_bad, my_bad);
    __syncthreads();
    if (j == 0 && n_bad) atomicAdd(bad_words, (unsigned long long)n_bad);
  }
}

__global__ void k_zero_u64(unsigned long long* p) { *p = 0; }

}  // namespace
}  // namespace mrl

extern "C" int mrl_thl_word_align(const float* src_logp, const uint8_t* src_mask,
                                  const int32_t* src_word_map, const int32_t* src_map_len,
                                  const uint8_t* tgt_mask, const int32_t* tgt_word_map,
                                  const int32_t* tgt_map_len, int64_t B, int32_t S_src, int32_t S_tgt,
                                  int32_t max_words, float ignore_value, float* out,
                                  int64_t* out_bad_words, void* stream) {
  using namespace mrl;
  if (B < 0 || S_src <= 0 || S_tgt <= 0 || B > ((int64_t)1 << 31) - 1) return MRL_ERR_SHAPE;
  if (max_words <= 0 || max_words > THL_MAX_WORDS) return MRL_ERR_SHAPE;
  if (B == 0) return MRL_OK;
  if (!src_logp || !src_mask || !src_word_map || !src_map_len || !tgt_mask || !tgt_word_map ||
      !tgt_map_len || !out)
    return MRL_ERR_NULL;
  const int rc = require_gfx950();
  if (rc != MRL_OK) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t lds = (size_t)max_words * 12;
  static LdsLimit lds_limit, lds_limit_short;
  static LdsLimit lds_limit_kept;
  lds_limit.ensure(reinterpret_cast<const void*>(&k_thl_word_align<false>), THL_MAX_WORDS * 12);
  lds_limit_kept.ensure(reinterpret_cast<const void*>(&k_thl_word_align<true>), THL_MAX_WORDS * 12);
  lds_limit_short.ensure(reinterpret_cast<const void*>(&k_thl_word_align_short), THL_MAX_WORDS * 12);
  const int longest = S_src > S_tgt ? S_src : S_tgt, words = max_words < THL_THREADS ? max_words : THL_THREADS;
  const bool is_short = longest <= THL_THREADS, is_kept = longest > THL_KEPT_FROM && longest <= THL_KEPT * THL_THREADS;
  const unsigned threads = is_short ? (unsigned)(((longest > words ? longest : words) + 63) / 64 * 64) : (unsigned)THL_THREADS;
  if (out_bad_words) hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(1), 0, s, reinterpret_cast<unsigned long long*>(out_bad_words));
  hipLaunchKernelGGL(is_short ? k_thl_word_align_short : is_kept ? k_thl_word_align<true> : k_thl_word_align<false>, dim3((unsigned)B), dim3(threads), lds, s, src_logp, src_mask,
                     src_word_map, src_map_len, tgt_mask, tgt_word_map, tgt_map_len, S_src, S_tgt, max_words,
                     ignore_value, out, reinterpret_cast<unsigned long long*>(out_bad_words));
  return hipGetLastError() == hipSuccess ? MRL_OK : MRL_ERR_DEVICE;
}
