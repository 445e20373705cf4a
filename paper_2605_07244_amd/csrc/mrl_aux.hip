// Memory-bound kernels of the scoring path: mask compaction, sequence weights,
// target logits, partial-merge + token-loss epilogue (Eq. 1 / Eq. 2 terms), operand
// preparation, the fp32 path's logits -> dz conversion, final reductions.
#include "mrl_finalize.h"
#include "mrl_internal.h"

namespace mrl {
namespace {

__device__ inline bool slot_valid(const uint8_t* mask, const int32_t* targets, int64_t n, int V) {
  const bool m = mask == nullptr || mask[n] != 0;
  const int32_t y = targets[n];
  return m && y >= 0 && y < V;
}

__device__ inline int valid_rows(const int64_t* n_scored, int64_t chunk_start, int chunk_rows) {
  const int64_t r = *n_scored - chunk_start;
  return r < 0 ? 0 : (r > chunk_rows ? chunk_rows : (int)r);
}

// ----------------------------------------------------------------------------
// Compaction of scored slots (order preserving), zeros in the per-slot outputs of the others, and
// the scored length of every sequence.  A launch that does next to nothing takes 4.5 - 5 us here,
// which the preparation of a small call is made of, so independent pieces share a launch: up to
// kPrepInline slots they are part of the row preparation (below); up to
// kPrepOneBlock slots one block compacts (and the other blocks of the launch count the sequences);
// above, one launch counts per block of slots (and per sequence) and one places the slots, each
// block adding up the counts before its own - up to kPrepMaxSelf blocks, beyond which a scan launch
// in between is cheaper than every block reading them all.
// As launches of their own count, scan, fill, sequence lengths and the zeros took 19 us before a loss call of 512 slots; the
// one launch takes 5.6 us for 3003 slots.
// ----------------------------------------------------------------------------
constexpr int PREP_PER_THREAD = 4;
constexpr int PREP_BLOCK = 256;
constexpr int PREP_PER_BLOCK = PREP_PER_THREAD * PREP_BLOCK;
constexpr int kPrepThreads = 1024;
constexpr int kPrepWaves = kPrepThreads / 64;
constexpr int64_t kPrepOneBlock = 32 * kPrepThreads;    // one bit per slot of a thread in a 32-bit word
constexpr int64_t kPrepMaxSelf = 4096;

struct SlotOutputs { float* o[3]; };                    // per-slot outputs that are 0 for unscored slots (or nullptr)
__device__ inline void zero_slot(const SlotOutputs& z, int64_t n) {
#pragma unroll
  for (int k = 0; k < 3; ++k) if (z.o[k] != nullptr) z.o[k][n] = 0.f;
}

__device__ inline int block_exclusive_scan(int val, int* total) {
  // 256 threads; returns the exclusive prefix of val, *total = block sum.
  __shared__ int wave_sums[4];
  __shared__ int wave_off[5];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = val;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int up = __shfl_up(incl, off);
    if (lane >= off) incl += up;
  }
  if (lane == 63) wave_sums[wave] = incl;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int w = 0; w < 4; ++w) { wave_off[w] = run; run += wave_sums[w]; }
    wave_off[4] = run;
  }
  __syncthreads();
  *total = wave_off[4];
  const int res = wave_off[wave] + incl - val;
  __syncthreads();
  return res;
}

// Scored slots of the sequences, by blocks of WAVES waves: a wave per sequence, or the block together where a
// sequence is long, since a wave alone is a chain of T / 256 load latencies.  Loss call of one sequence of 32768 slots
// (V = 64, d = 8) 817 us by waves, now 707, two of 10^6 slots, 500 scored (V = 1000, d = 64) 5740 and 1930.
constexpr int kLongSequence = 1024;
template <int N> struct Stride { static constexpr int value = N; };
template <int WAVES> __device__ inline void count_sequences(const uint8_t* mask, const int32_t* targets, int64_t block,
                                                            int64_t B, int T, int V, int32_t* seq_len) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto wave_count = [&](int64_t b, int first, auto stride) {
    int cnt = 0;
#pragma unroll 4
    for (int t = first; t < T; t += decltype(stride)::value) cnt += slot_valid(mask, targets, b * T + t, V);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
    return cnt;
  };
  if (T > kLongSequence) {
    __shared__ int part[WAVES];
    const int cnt = wave_count(block, threadIdx.x, Stride<64 * WAVES>{});
    if (lane == 0) part[wave] = cnt;
    __syncthreads();
    if (threadIdx.x != 0) return;
    int sum = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) sum += part[w];
    seq_len[block] = sum;
  } else if (block * WAVES + wave < B) {
    const int cnt = wave_count(block * WAVES + wave, lane, Stride<64>{});
    if (lane == 0) seq_len[block * WAVES + wave] = cnt;
  }
}
// blocks the above takes
inline int64_t sequence_blocks(int64_t B, int T, int waves) { return T > kLongSequence ? B : (B + waves - 1) / waves; }

// Row copy with zero padding: out[r][0:dp] = in[r][0:d] | 0, for a W whose width is no multiple of the forward
// kernel's 128-wide panel pairs: its last 128 columns, or all of it where it is narrower than that or its
// rows are no whole lines and the pass is long (head_tail_only in mrl_api.hip).
constexpr int PAD_VECTORS = 4;                          // 16-byte vectors per thread
template <int THREADS> __device__ inline void pad_rows(const PadRows& p, int64_t block) {
  const int per_row = p.dp / 8;
#pragma unroll
  for (int k = 0; k < PAD_VECTORS; ++k) {
    const int64_t i = (block * PAD_VECTORS + k) * THREADS + threadIdx.x;
    const int64_t r = i / per_row;
    if (r >= p.rows) return;
    const int c = (int)(i - r * per_row) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (c < p.d) v = *reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(p.in) + r * p.ld_in + c);
    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(p.out) + r * p.ld_out + c) = v;
  }
}
inline int64_t pad_blocks(const PadRows& p, int threads) {
  const int64_t per_block = PAD_VECTORS * threads;
  return (p.rows * (p.dp / 8) + per_block - 1) / per_block;
}
__global__ __launch_bounds__(256) void k_pad_rows_b16(PadRows p) { pad_rows<256>(p, blockIdx.x); }

// Block 0: N <= kPrepOneBlock slots, a contiguous run of them per wave.  The blocks behind it: the sequences, up to first_pad, and the padded
// columns of W, if there are any (a launch of their own: scoring call of 3003 slots, V = 50257, d = 712 158 us, now 153).
__global__ __launch_bounds__(kPrepThreads) void k_prep_one(const uint8_t* mask, const int32_t* targets, int N, int V,
                                                           int64_t* n_scored, int64_t* n_bad, int32_t* row_index,
                                                           SlotOutputs zero, int64_t B, int T, int32_t* seq_len, PadRows pad, int first_pad) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if ((int)blockIdx.x >= first_pad) { pad_rows<kPrepThreads>(pad, (int64_t)blockIdx.x - first_pad); return; }
  if (blockIdx.x > 0) {
    count_sequences<kPrepWaves>(mask, targets, (int64_t)blockIdx.x - 1, B, T, V, seq_len);
    return;
  }
  __shared__ int sums[kPrepWaves], bads[kPrepWaves];
  const int iters = (N + kPrepThreads - 1) / kPrepThreads;
  const int first = wave * iters * 64;
  uint32_t bits = 0;
  int cnt = 0, bad = 0;
#pragma unroll 8
  for (int it = 0; it < iters; ++it) {
    const int n = first + it * 64 + lane;
    bool scored = false, ok = false;
    if (n < N) {
      const int32_t y = targets[n];
      ok = y >= 0 && y < V;
      scored = mask == nullptr || mask[n] != 0;
    }
    bits |= (uint32_t)(scored && ok) << it;
    cnt += scored && ok;
    bad += scored && !ok;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) { cnt += __shfl_xor(cnt, off); bad += __shfl_xor(bad, off); }
  if (lane == 0) { sums[wave] = cnt; bads[wave] = bad; }
  __syncthreads();
  int pos = 0, total = 0, total_bad = 0;
#pragma unroll
  for (int w = 0; w < kPrepWaves; ++w) {
    pos += w < wave ? sums[w] : 0;
    total += sums[w];
    total_bad += bads[w];
  }
  if (threadIdx.x == 0) { *n_scored = total; *n_bad = total_bad; }
  for (int it = 0; it < iters; ++it) {
    const int n = first + it * 64 + lane;
    const bool ok = (bits >> it) & 1;
    const unsigned long long ball = __ballot(ok);
    if (ok) row_index[pos + __popcll(ball & ((1ull << lane) - 1ull))] = n;
    else if (n < N) zero_slot(zero, n);
    pos += __popcll(ball);
    if (n < N && n >= total) row_index[n] = 0;          // tail entries: a harmless valid slot
  }
}

// Blocks below nblocks: counts of their slots.  Blocks from nblocks on: the sequences.
__global__ __launch_bounds__(PREP_BLOCK) void k_prep_count(const uint8_t* mask, const int32_t* targets,
                                                          int64_t N, int V, int32_t* block_counts,
                                                          int64_t nblocks, int64_t B, int T, int32_t* seq_len) {
  if (blockIdx.x >= nblocks) {
    count_sequences<PREP_BLOCK / 64>(mask, targets, (int64_t)blockIdx.x - nblocks, B, T, V, seq_len);
    return;
  }
  const int64_t base = (int64_t)blockIdx.x * PREP_PER_BLOCK + threadIdx.x * PREP_PER_THREAD;
  int cnt = 0, bad = 0;
#pragma unroll
  for (int k = 0; k < PREP_PER_THREAD; ++k) {
    const int64_t n = base + k;
    if (n < N) {
      const bool m = mask == nullptr || mask[n] != 0;
      const int32_t y = targets[n];
      const bool ok = y >= 0 && y < V;
      cnt += (m && ok);
      bad += (m && !ok);
    }
  }
  int tot_c, tot_b;
  block_exclusive_scan(cnt, &tot_c);
  block_exclusive_scan(bad, &tot_b);
  if (threadIdx.x == 0) {
    block_counts[blockIdx.x] = tot_c;
    block_counts[nblocks + blockIdx.x] = tot_b;
  }
}

__global__ __launch_bounds__(1024) void k_prep_scan(int32_t* block_counts, int64_t nblocks,
                                                   int64_t* block_offsets, int64_t* n_scored,
                                                   int64_t* n_bad) {
  // single block: exclusive scan of block_counts[0..nblocks) into block_offsets (int64)
  __shared__ int64_t sh[1024];
  __shared__ int64_t carry, bad_total;
  if (threadIdx.x == 0) { carry = 0; bad_total = 0; }
  __syncthreads();
  for (int64_t base = 0; base < nblocks; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int64_t v = i < nblocks ? block_counts[i] : 0;
    const int64_t b = i < nblocks ? block_counts[nblocks + i] : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
      const int64_t t = threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
      __syncthreads();
      sh[threadIdx.x] += t;
      __syncthreads();
    }
    if (i < nblocks) block_offsets[i] = carry + sh[threadIdx.x] - v;
    __syncthreads();
    const int64_t chunk_total = sh[1023];
    // reuse sh for the bad-target sum
    __syncthreads();
    sh[threadIdx.x] = b;
    __syncthreads();
    for (int off = 512; off > 0; off >>= 1) {
      if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
      __syncthreads();
    }
    if (threadIdx.x == 0) { carry += chunk_total; bad_total += sh[0]; }
    __syncthreads();
  }
  if (threadIdx.x == 0) { *n_scored = carry; *n_bad = bad_total; }
}

// block_offsets == nullptr: the block adds up the counts itself, and block 0 publishes the totals
__global__ __launch_bounds__(PREP_BLOCK) void k_prep_fill(const uint8_t* mask, const int32_t* targets,
                                                         int64_t N, int V, const int32_t* block_counts, int64_t nblocks,
                                                         const int64_t* block_offsets, int64_t* n_scored,
                                                         int64_t* n_bad, int32_t* row_index, SlotOutputs zero) {
  const int64_t base = (int64_t)blockIdx.x * PREP_PER_BLOCK + threadIdx.x * PREP_PER_THREAD;
  bool ok[PREP_PER_THREAD];
  int cnt = 0;
#pragma unroll
  for (int k = 0; k < PREP_PER_THREAD; ++k) {
    const int64_t n = base + k;
    ok[k] = n < N && slot_valid(mask, targets, n, V);
    cnt += ok[k];
  }
  int64_t before, ns;
  if (block_offsets == nullptr) {
    // (kPrepMaxSelf blocks of 1024 slots: the sums fit 32 bits)
    int own = 0, all = 0, bad = 0, sum_own, sum_all, sum_bad;
#pragma unroll 4
    for (int i = threadIdx.x; i < nblocks; i += PREP_BLOCK) {
      const int c = block_counts[i];
      all += c;
      own += i < blockIdx.x ? c : 0;
      if (blockIdx.x == 0) bad += block_counts[nblocks + i];
    }
    block_exclusive_scan(own, &sum_own);
    block_exclusive_scan(all, &sum_all);
    before = sum_own;
    ns = sum_all;
    if (blockIdx.x == 0) {
      block_exclusive_scan(bad, &sum_bad);
      if (threadIdx.x == 0) { *n_scored = sum_all; *n_bad = sum_bad; }
    }
  } else {
    before = block_offsets[blockIdx.x];
    ns = *n_scored;
  }
  int total;
  const int excl = block_exclusive_scan(cnt, &total);
  int64_t pos = before + excl;
#pragma unroll
  for (int k = 0; k < PREP_PER_THREAD; ++k) {
    const int64_t n = base + k;
    if (ok[k]) row_index[pos++] = (int32_t)n;
    else if (n < N) zero_slot(zero, n);
    if (n < N && n >= ns) row_index[n] = 0;   // tail entries: a harmless valid slot
  }
}

// ----------------------------------------------------------------------------
// The aggregation weights of Eq. (1) / Eq. (2): one block.
// ----------------------------------------------------------------------------
constexpr int kCoefLdsGroups = 4096;
__device__ inline void block_sum3(long long (&v)[3], long long (*sh)[3]) {   // 256 threads; the sums in every thread
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off);
  __syncthreads();
  if ((threadIdx.x & 63) == 0)
    for (int k = 0; k < 3; ++k) sh[threadIdx.x >> 6][k] = v[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 3; ++k) v[k] = sh[0][k] + sh[1][k] + sh[2][k] + sh[3][k];
}

struct CoefArgs {
  const int32_t* seq_len; const int32_t* group_id; const uint8_t* seq_kind; int64_t B; int G; int loss_agg;
  int32_t* group_count; float* seq_coef; int64_t* n_bad_groups;
};
// f(sequence, live, kind, scored length, group id or -1, of_group(group id)) for the block's sequences, the loads of
// STEPS of them in flight together: one after the other they cost the single block 0.2 us per 256 sequences and
// loop.  Steps beyond the last sequence see that one again, not live, and f has no branches: with one per
// step the kernel needed 100 scalar registers, and the blocks that clear dH rows had fewer waves in flight (2^20 slots,
// 500 scored, d = 64: 421 us a call, now 373).  Loss call of 65536 sequences of one token, V = 1024, d = 128: 8192
// groups 1494 us one at a time, now 1316, 60000 groups 1559 and 1349.
constexpr int kCoefSteps = 4;
template <int STEPS, class Of, class F> __device__ inline void each_sequence(const CoefArgs& a, Of of_group, F f) {
  for (int64_t b0 = threadIdx.x; b0 < a.B; b0 += 256 * STEPS) {
    int kind[STEPS], len[STEPS], group[STEPS], of[STEPS];
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
      const int64_t b = b0 + 256 * k < a.B ? b0 + 256 * k : a.B - 1;
      kind[k] = a.seq_kind ? a.seq_kind[b] : 0;
      len[k] = a.seq_len[b];
      group[k] = a.group_id[b];
    }
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
      group[k] = group[k] >= 0 && group[k] < a.G ? group[k] : -1;
      of[k] = of_group(group[k] < 0 ? 0 : group[k]);
    }
#pragma unroll
    for (int k = 0; k < STEPS; ++k) {
      const bool live = b0 + 256 * k < a.B;
      f(live ? b0 + 256 * k : a.B - 1, live, kind[k], len[k], group[k], of[k]);
      __builtin_amdgcn_sched_barrier(0);              // (interleaved, they would keep their masks alive together)
    }
  }
}
template <int STEPS>
__device__ inline void seq_coef_block(const CoefArgs& a, int32_t* lds_count /*[kCoefLdsGroups]*/) {
  __shared__ long long sh[4][3];
  const bool in_lds = a.G <= kCoefLdsGroups;
  // group counts: in LDS, or with device-scope atomics in global memory
  auto count = [&](int g) { return in_lds ? lds_count[g] : __hip_atomic_load(&a.group_count[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  for (int g = threadIdx.x; g < a.G; g += 256) {
    if (in_lds) lds_count[g] = 0;
    else __hip_atomic_store(&a.group_count[g], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __threadfence();
  __syncthreads();
  long long v[3] = {0, 0, 0};                         // auxiliary rows with tokens, GRPO tokens, bad group ids
  each_sequence<STEPS>(a, [](int) { return 0; }, [&](int64_t, bool live, int kind, int L, int g, int) {
    const bool grpo = live && kind == 0 && g >= 0;
    v[0] += live && kind != 0 && L > 0;
    v[1] += grpo ? L : 0;
    v[2] += live && g < 0;
    const int at = g < 0 ? 0 : g;
    if (in_lds) atomicAdd(&lds_count[at], (int)grpo); else atomicAdd(&a.group_count[at], (int)grpo);
  });
  __threadfence();
  block_sum3(v, sh);                                  // (its barriers also publish the counts)
  long long u[3] = {0, 0, 0};
  for (int g0 = threadIdx.x; g0 < a.G; g0 += 256 * STEPS) {
    int n[STEPS];
#pragma unroll
    for (int k = 0; k < STEPS; ++k) n[k] = count(g0 + 256 * k < a.G ? g0 + 256 * k : a.G - 1);
#pragma unroll
    for (int k = 0; k < STEPS; ++k) u[0] += g0 + 256 * k < a.G && n[k] > 0;
  }
  block_sum3(u, sh);
  if (threadIdx.x == 0) *a.n_bad_groups = v[2];
  const double P = (double)u[0], S = (double)v[0], NT = (double)v[1];
  each_sequence<STEPS>(a, count, [&](int64_t b, bool, int kind, int L, int g, int K) {
    const double mean = (kind == 0 ? P * (double)K : S) * (double)L;
    const double weight = 1.0 / (kind == 0 && a.loss_agg == 1 ? NT : mean);
    a.seq_coef[b] = L > 0 && (kind != 0 || g >= 0) ? (float)weight : 0.f;   // (the last sequence: the same from all)
  });
}

// ----------------------------------------------------------------------------
// Response-level log-ratio: one workgroup per sequence, fp64 partial sums, fixed order.
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_seq_log_ratio(const uint8_t* mask, const int32_t* targets,
                                                       const float* logp, const float* behav, int T, int V,
                                                       int level, float* seq_expo) {
  __shared__ double sh[256];
  __shared__ int shn[256];
  const int64_t b = blockIdx.x;
  double acc = 0.0;
  int cnt = 0;
  for (int t = threadIdx.x; t < T; t += 256) {
    const int64_t n = b * T + t;
    if (slot_valid(mask, targets, n, V)) { acc += (double)logp[n] - (double)behav[n]; ++cnt; }
  }
  sh[threadIdx.x] = acc;
  shn[threadIdx.x] = cnt;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) { sh[threadIdx.x] += sh[threadIdx.x + off]; shn[threadIdx.x] += shn[threadIdx.x + off]; }
    __syncthreads();
  }
  if (threadIdx.x == 0) seq_expo[b] = (float)(level == 2 ? (shn[0] > 0 ? sh[0] / shn[0] : 0.0) : sh[0]);
}

// ----------------------------------------------------------------------------
// Row preparation: what needs the compaction and comes before a forward launch, in one launch.
//   one block (PREP)    : the compaction's outputs
//   one block (loss)    : with PREP the scored lengths, and the sequence weights
//   zero_blocks         : dH rows of unscored slots, ZERO_SLOTS_PER_BLOCK each
//   the rest            : one wave per scored row of the pass: target logit z_t = <H[slot], W[y]> and,
//                         on the bf16 path, the row's copy Hc[r][0:dp] = H[slot][0:d] | 0, which
//                         gives the forward launch contiguous rows (no index lookups in that kernel)
//                         and a K extent that is a multiple of its 128-wide panel pairs
// As launches of their own the pieces took 37 us before the forward launch of 512 slots (now 12), and the
// target logits read the hidden rows a second time.
// ----------------------------------------------------------------------------
constexpr int ZERO_SLOTS_PER_BLOCK = 16;
__device__ inline float bf16_bits_to_float(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

__device__ inline void zero_dh_rows(const RowPrepArgs& a, int64_t first) {
  for (int s = 0; s < ZERO_SLOTS_PER_BLOCK; ++s) {
    const int64_t n = first + s;
    if (n >= a.N) return;
    if (slot_valid(a.mask, a.targets, n, a.V)) continue;
    unsigned char* row = static_cast<unsigned char*>(a.dH) + n * a.dh_row_bytes;
    if ((a.dh_row_bytes & 15) == 0 && (reinterpret_cast<uintptr_t>(a.dH) & 15) == 0) {
      const uint4 z = make_uint4(0, 0, 0, 0);
      for (int64_t o = threadIdx.x * 16; o < a.dh_row_bytes; o += 256 * 16) *reinterpret_cast<uint4*>(row + o) = z;
    } else {
      for (int64_t o = threadIdx.x * 4; o < a.dh_row_bytes; o += 256 * 4) *reinterpret_cast<uint32_t*>(row + o) = 0u;
    }
  }
}

// Compaction of N <= kPrepInline slots by one block of 256: a contiguous run of slots per wave, f(slot, rank among the scored
// ones, scored, masked in with a bad target) per slot; returns the number of scored ones.  Every block of the
// launch that needs it does it for itself (10 KB from the L2), which takes less than a launch that does it once.
template <class F>
__device__ inline int compact_block(const uint8_t* mask, const int32_t* targets, int N, int V, F f) {
  constexpr int kIters = kPrepInline / 256;
  __shared__ int sums[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int iters = (N + 255) / 256, first = wave * iters * 64;
  uint32_t scored = 0, bad = 0;
  int cnt = 0;
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    const int n = first + it * 64 + lane;
    if (it < iters && n < N) {
      const int32_t y = targets[n];
      const bool in = mask == nullptr || mask[n] != 0, ok = y >= 0 && y < V;
      scored |= (uint32_t)(in && ok) << it;
      bad |= (uint32_t)(in && !ok) << it;
    }
  }
#pragma unroll
  for (int it = 0; it < kIters; ++it) cnt += __popcll(__ballot((scored >> it) & 1));
  if (lane == 0) sums[wave] = cnt;
  __syncthreads();
  int pos = 0, total = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) { pos += w < wave ? sums[w] : 0; total += sums[w]; }
#pragma unroll
  for (int it = 0; it < kIters; ++it) {
    const int n = first + it * 64 + lane;
    const bool ok = (scored >> it) & 1;
    const unsigned long long ball = __ballot(ok);
    if (it < iters && n < N) f(n, pos + __popcll(ball & ((1ull << lane) - 1ull)), ok, ((bad >> it) & 1) != 0);
    pos += __popcll(ball);
  }
  return total;
}

// PREP: what k_prep_one does comes with this launch
template <bool BF16, bool PREP>
__global__ __launch_bounds__(256) void k_row_prep(RowPrepArgs a, PrepOut prep) {
  __shared__ int32_t lds_count[kCoefLdsGroups];
  int64_t block = blockIdx.x;
  if (PREP) {
    if (block == 0) {
      // the compaction's outputs
      int bad = 0;
      const int N = (int)a.N;
      const SlotOutputs zero = {{prep.zero[0], prep.zero[1], prep.zero[2]}};
      const int total = compact_block(a.mask, a.targets, N, a.V, [&](int n, int rank, bool ok, bool wrong) {
        if (ok) prep.row_index[rank] = n;
        else zero_slot(zero, n);
        bad += wrong;
      });
      for (int n = total + threadIdx.x; n < N; n += 256) prep.row_index[n] = 0;     // tail entries: a harmless valid slot
      __shared__ int bads[4];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off);
      if ((threadIdx.x & 63) == 0) bads[threadIdx.x >> 6] = bad;
      __syncthreads();
      if (threadIdx.x == 0) { *prep.n_scored = total; *prep.n_bad = bads[0] + bads[1] + bads[2] + bads[3]; }
      return;
    }
    --block;
  }
  if (a.seq_coef != nullptr) {
    if (block == 0) {
      if (PREP) {
        // scored slots of the sequences (B <= N <= kPrepInline)
        static_assert(kPrepInline <= kCoefLdsGroups, "a count per sequence");
        for (int b = threadIdx.x; b < prep.B; b += 256) lds_count[b] = 0;
        __syncthreads();
        for (int n = threadIdx.x; n < (int)a.N; n += 256)
          if (slot_valid(a.mask, a.targets, n, a.V)) atomicAdd(&lds_count[n / prep.T], 1);
        __syncthreads();
        for (int b = threadIdx.x; b < prep.B; b += 256) prep.seq_len[b] = lds_count[b];
        __threadfence_block();
        __syncthreads();
      }
      const CoefArgs c = {a.seq_len, a.group_id, a.seq_kind, a.B, a.G, a.loss_agg, a.group_count, a.seq_coef, a.n_bad_groups};
      if (a.B <= 256) seq_coef_block<1>(c, lds_count); else seq_coef_block<kCoefSteps>(c, lds_count);
      return;
    }
    --block;
  }
  if (block < a.zero_blocks) { zero_dh_rows(a, block * ZERO_SLOTS_PER_BLOCK); return; }
  block -= a.zero_blocks;
  const int64_t r = block * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  int64_t slot;
  if (PREP) {
    __shared__ int32_t slots[4];
    const int r0 = (int)(a.chunk_start + block * 4);  // (rank of the block's first row)
    if (r0 >= (int)a.N) return;
    const int total = compact_block(a.mask, a.targets, (int)a.N, a.V, [&](int n, int rank, bool ok, bool) {
      if (ok && rank >= r0 && rank < r0 + 4) slots[rank - r0] = n;
    });
    __syncthreads();
    if (r >= a.chunk_rows || a.chunk_start + r >= total) return;
    slot = slots[threadIdx.x >> 6];
  } else {
    if (r >= valid_rows(a.n_scored, a.chunk_start, a.chunk_rows)) return;
    slot = a.row_index[a.chunk_start + r];
  }
  const int64_t y = a.targets[slot];
  float acc = 0.f;
  if (BF16) {
    const uint4* h = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.H) + slot * a.d);
    const uint4* w = reinterpret_cast<const uint4*>(static_cast<const uint16_t*>(a.W) + y * a.d);
    // the row's vectors, side by side or in blocks of kRowBlock columns
    const bool blocks = rows_in_blocks(a.chunk_rows);
    uint4* const out = static_cast<uint4*>(a.Hc) + r * (blocks ? kRowBlock / 8 : a.ldh / 8);
    const int64_t block_step = (int64_t)a.chunk_rows * (kRowBlock / 8);
    auto at = [&](int c) { return blocks ? c / (kRowBlock / 8) * block_step + c % (kRowBlock / 8) : c; };
#pragma unroll 4
    for (int c = lane; c < a.d / 8; c += 64) {
      const uint4 u = h[c], b = w[c];
      out[at(c)] = u;
      const uint32_t av[4] = {u.x, u.y, u.z, u.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        acc = fmaf(bf16_bits_to_float(av[q] & 0xffffu), bf16_bits_to_float(bv[q] & 0xffffu), acc);
        acc = fmaf(bf16_bits_to_float(av[q] >> 16), bf16_bits_to_float(bv[q] >> 16), acc);
      }
    }
    for (int c = a.d / 8 + lane; c < a.dp / 8; c += 64) out[at(c)] = make_uint4(0, 0, 0, 0);
  } else {
    const float* h = static_cast<const float*>(a.H) + slot * a.d;
    const float* w = static_cast<const float*>(a.W) + y * a.d;
    for (int c = lane; c < a.d; c += 64) acc = fmaf(h[c], w[c], acc);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (lane == 0) a.zt[a.chunk_start + r] = acc;
}

// ----------------------------------------------------------------------------
// fp32 path: one (max, sum-exp) partial per row of the materialised chunk logits.
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_row_lse_f32(const float* Z, int64_t ldz, const int64_t* n_scored,
                                                     int64_t chunk_start, int chunk_rows, int V,
                                                     float* part_max, float* part_sum, float* part_ez) {
  const int i = blockIdx.x;
  if (i >= valid_rows(n_scored, chunk_start, chunk_rows)) return;
  __shared__ float sh[256];
  const float* z = Z + (int64_t)i * ldz;
  float mx = -INFINITY;
  for (int v = threadIdx.x; v < V; v += 256) mx = fmaxf(mx, z[v]);
  sh[threadIdx.x] = mx;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) sh[threadIdx.x] = fmaxf(sh[threadIdx.x], sh[threadIdx.x + off]);
    __syncthreads();
  }
  mx = sh[0];
  __syncthreads();
  float s = 0.f;
  for (int v = threadIdx.x; v < V; v += 256) s += expf(z[v] - mx);
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) { part_max[i] = mx; part_sum[i] = sh[0]; }
  if (part_ez == nullptr) return;
  __syncthreads();
  float t = 0.f;
  for (int v = threadIdx.x; v < V; v += 256) t += expf(z[v] - mx) * z[v];
  sh[threadIdx.x] = t;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part_ez[i] = sh[0];
}

// ----------------------------------------------------------------------------
// Row epilogue: merge partials -> lse, log-prob; Eq. (1) token terms; loss partials; for the
// bf16 backward the row scale -g / S and the patch of the stash's target column.
// Block = 64 rows x 64 partial lanes: a thread adds every 64th partial of 4 neighbouring rows (16-byte
// loads, eight in flight, the last batch as long as the power of two that takes what is left: V = 50257 has 394 partials, seven per thread, which
// the remainder of a loop unrolled by eight took one latency after the other), so that a pass of few rows is not a chain of hundreds of dependent-latency
// loads (with 4 lanes per row: 112 us for 1188 partials and 201 rows; now 9 us, and 72 us instead of 150
// for 65536 rows, whose partials are 311 MB).
// ----------------------------------------------------------------------------
constexpr int EPI_ROWS = 64;
constexpr int EPI_THREADS = 1024;
constexpr int EPI_LANES = EPI_THREADS / (EPI_ROWS / 4);
// K loads of a thread's partials, in flight together: every EPI_LANES-th from q on, of which `left` (of the block's numbering) remain.
template <int K, bool ALL> __device__ __forceinline__ void add_partials(const float* q, int64_t step, int left, float4& s) {
  float4 v[K];
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = *reinterpret_cast<const float4*>(ALL || k * EPI_LANES < left ? q + k * step : q);
#pragma unroll
  for (int k = 0; k < K; ++k)
    if (ALL || k * EPI_LANES < left) { s.x += v[k].x; s.y += v[k].y; s.z += v[k].z; s.w += v[k].w; }
}
// Sum over all partials of this block's 64 rows; the result is valid in threads 0 .. 63 (one row
// each).  Fixed order.  src points at the block's first row; rows beyond the valid ones hold
// whatever the buffer held.  All threads must call it.
__device__ inline float merge_partials(const float* src, int64_t stride, int n_partials, float4 (&sh)[EPI_LANES][EPI_ROWS / 4]) {
  const int quad = threadIdx.x & 15, part = threadIdx.x >> 4;
  const int64_t step = stride * EPI_LANES;
  const float* q = src + (part < n_partials ? part : 0) * stride + quad * 4;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  int rest = n_partials;                              // from the block's first on
  for (; rest >= EPI_LANES * 8; rest -= EPI_LANES * 8, q += 8 * step) add_partials<8, true>(q, step, 0, s);
  const int left = rest - part;                       // the thread's first is `part` of them
  if (rest > EPI_LANES * 4) add_partials<8, false>(q, step, left, s);
  else if (rest > EPI_LANES * 2) add_partials<4, false>(q, step, left, s);
  else if (rest > EPI_LANES) add_partials<2, false>(q, step, left, s);
  else if (left > 0) add_partials<1, true>(q, step, 0, s);
  __syncthreads();                                  // an earlier merge has been read
  sh[part][quad] = s;
  __syncthreads();
  // 16 waves, one row per lane, 4 lanes' sums each; then the 16 wave sums by the first wave
  const int row = threadIdx.x & 63, wave = threadIdx.x >> 6;
  auto cell = [&](int l) -> float& { return reinterpret_cast<float*>(&sh[l][0])[row]; };
  const float t = (cell(4 * wave) + cell(4 * wave + 1)) + (cell(4 * wave + 2) + cell(4 * wave + 3));
  __syncthreads();
  cell(wave) = t;
  __syncthreads();
  float sum = 0.f;
  if (wave == 0) {
#pragma unroll
    for (int w = 0; w < EPI_THREADS / 64; ++w) sum += cell(w);
  }
  return sum;
}

// Eq. (1) / Eq. (2) terms of a scored token: returns dL/dl and sets the token's entries of the loss partials.
__device__ __forceinline__ float token_terms(const RowEpiArgs& a, int64_t slot, float logp, double (&q)[EPI_NQ]) {
  const int64_t b = slot / a.T;
  const float c = a.seq_coef[b];
  const int kind = a.seq_kind ? a.seq_kind[b] : 0;
  if (kind != 0) {
    q[2] = -(double)c * (double)logp;
    return -a.lambda * c;
  }
  const float A = a.seq_adv[b];
  // token ratio of Eq. (1), or the response's ratio (App. I.1) whose derivative with
  // respect to each token's log-prob is rho (summed form) or rho / L_b (mean form)
  const float w = a.seq_expo ? expf(a.seq_expo[b]) : expf(logp - a.behav_logp[slot]);
  const float s1 = w * A;
  const float wc = fminf(fmaxf(w, 1.f - a.eps_lo), 1.f + a.eps_hi);
  const float s2 = wc * A;
  const float J = fminf(s1, s2);
  float dJ = s1 <= s2 ? s1 : 0.f;
  if (a.seq_expo && a.ratio_level == 1) dJ *= (float)a.seq_len[b];
  float k3 = 0.f, dk3 = 0.f;
  if (a.ref_logp != nullptr) {
    const float rho = a.ref_logp[slot] - logp;
    const float em1 = expm1f(rho);
    k3 = em1 - rho;
    dk3 = -em1;
  }
  q[0] = -(double)c * (double)J;
  q[1] = (double)c * (double)k3;
  q[3] = (double)w;
  q[4] = w > 0.f ? (double)w : 0.0;            // (a NaN ratio is left out of the maximum)
  q[5] = (double)k3;
  q[6] = (w < 1.f - a.eps_lo || w > 1.f + a.eps_hi) ? 1.0 : 0.0;
  q[7] = s2 < s1 ? 1.0 : 0.0;
  q[8] = 1.0;
  return c * (-dJ + a.beta * dk3);
}

__global__ __launch_bounds__(EPI_THREADS) void k_row_epilogue(RowEpiArgs a) {
  __shared__ float4 sh[EPI_LANES][EPI_ROWS / 4];
  const int nvalid = valid_rows(a.n_scored, a.chunk_start, a.chunk_rows);
  const int r0 = blockIdx.x * EPI_ROWS;               // first row of the block within the chunk
  const int tx = threadIdx.x & 63;
  const int i = r0 + tx;
  const bool live = i < nvalid;
  const bool offset_sums = a.part_max == nullptr;     // bf16 kernel: sums of 2^(z log2e - c2)
  if (r0 >= nvalid) {                                 // nothing here: an empty entry in the loss partials
    if (a.loss_partials != nullptr && threadIdx.x < EPI_NQ)
      a.loss_partials[(a.partial_block_offset + blockIdx.x) * EPI_NQ + threadIdx.x] = 0.0;
    return;
  }

  float s = 0.f, tsum = 0.f, mx = 0.f;
  if (offset_sums) {
    s = merge_partials(a.part_sum + r0, a.chunk_rows, a.n_partials, sh);
    if (a.part_ez != nullptr) tsum = merge_partials(a.part_ez + r0, a.chunk_rows, a.n_partials, sh);
  } else if (live) {                                  // fp32 path: one (max, sum-exp) pair per row
    s = a.part_sum[i];
    mx = a.part_max[i];
    if (a.part_ez != nullptr) tsum = a.part_ez[i];
  }
  if (threadIdx.x >= 64) return;                      // one thread per row from here on

  double q[EPI_NQ];
#pragma unroll
  for (int k = 0; k < EPI_NQ; ++k) q[k] = 0.0;
  if (live) {
    constexpr float LOG2E = 1.4426950408889634f;
    constexpr double LN2 = 0.6931471805599453;
    const int64_t ci = a.chunk_start + i;
    const float zt = a.zt[ci];
    // offset sums: lse = (c2 + log2 S) ln 2 with the very c2 the forward kernel subtracted
    const double lse_d = offset_sums ? ((double)fmaf(zt, LOG2E, kStashMargin2) + log2((double)s)) * LN2
                                     : (double)mx + log((double)s);
    const float lse = (float)lse_d;
    const float logp = (float)((double)zt - lse_d);
    const int64_t slot = a.row_index[ci];
    a.out_logp[slot] = logp;
    if (a.out_lse) a.out_lse[slot] = lse;
    if (a.lse_c) a.lse_c[ci] = lse;
    if (a.part_ez != nullptr) {
      // entropy H = lse - (sum_v e z) / (sum_v e)
      a.out_entropy[slot] = (float)(lse_d - (double)tsum / (double)s);
    }
    // A target log-prob below the range the bf16 backward operands represent (only possible for a
    // token the learner deems impossible): the row is counted and dropped from the loss and the
    // gradients (weight 0), as a row with an invalid target would be.
    const bool saturated = offset_sums && logp < kSaturatedLogp;
    if (saturated) {
      q[9] = 1.0;
      if (a.g_c) a.g_c[ci] = 0.f;
      if (a.row_scale) a.row_scale[ci] = 0.f;
    }
    if (a.seq_coef != nullptr && !saturated) {
      const float g = token_terms(a, slot, logp, q);
      if (a.g_c) a.g_c[ci] = g;
      if (a.row_scale) {
        // dz = g (onehot - e / S) = (-g / S) (e - S onehot): the scale, and the one entry of the
        // stash row that differs from e
        a.row_scale[ci] = -g / s;
        uint16_t* cell = a.estash + (int64_t)i * a.lde + a.targets[slot];
        const float e_y = __uint_as_float((uint32_t)*cell << 16);
        const __bf16 patched = (__bf16)(e_y - s);
        uint16_t bits;
        __builtin_memcpy(&bits, &patched, 2);
        *cell = bits;
      }
    }
  }
  if (a.loss_partials == nullptr) return;
  // fixed-order reduction over the block's 64 rows (one wave)
  double* out = a.loss_partials + (a.partial_block_offset + blockIdx.x) * EPI_NQ;
#pragma unroll
  for (int k = 0; k < EPI_NQ; ++k) q[k] = k == 4 ? wave_max64(q[k]) : wave_sum64(q[k]);
  if (tx == 0) {
#pragma unroll
    for (int k = 0; k < EPI_NQ; ++k) out[k] = q[k];
  }
}

// ----------------------------------------------------------------------------
// fp32 path, vocabularies of at most kRowLogits ids: log-sum-exp, row epilogue and conversion to dz in one launch, a wave per
// row, which keeps the row's logits in registers in between; 16 rows per block and entry of the loss partials.
// As three launches (a block per row, 64 rows per block, a grid of rows) they are three latencies of 4 - 5 us each
// on kilobytes (loss call of 256 slots, V = 512, d = 64, which the host bounds: 35.1 us, now 31.6).
// The loops over a lane's logits are unrolled, and what lies behind V costs its issue: two lengths.  Loss calls, us, of 232
// and of 20000 rows, d = 64, with loops of 2048 and of 512: V = 300 23.1 and 22.0, 473 and 462; V = 400 23.6 and 22.9, 495 and
// 486; V = 512 24.5 and 23.6, 513 and 507.  A third length, of 1024, would take 1 % off 513 to 1024 ids (V = 600 25.9 and 25.4,
// 526 and 521), and is not worth another instance; one in the place of 512 adds 0.5 % below that.
// ----------------------------------------------------------------------------
constexpr int kRowLogits = 2048, kFewLogits = 512, kRowWaves = 16;
template <int LOGITS>
__global__ __launch_bounds__(kRowWaves * 64) void k_row_f32(RowEpiArgs a, float* Z, int64_t ldz, int V, int write_dz) {
  __shared__ double sh[kRowWaves][EPI_NQ];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = blockIdx.x * kRowWaves + wave;
  double q[EPI_NQ];
#pragma unroll
  for (int k = 0; k < EPI_NQ; ++k) q[k] = 0.0;
  if (i < valid_rows(a.n_scored, a.chunk_start, a.chunk_rows)) {
    float* const row = Z + (int64_t)i * ldz;
    float z[LOGITS / 64];
    float mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < LOGITS / 64; ++k) {
      const int v = k * 64 + lane;
      z[k] = v < V ? row[v] : -INFINITY;
      mx = fmaxf(mx, z[k]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < LOGITS / 64; ++k)
      if (k * 64 < V) s += k * 64 + lane < V ? expf(z[k] - mx) : 0.f;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    const int64_t ci = a.chunk_start + i, slot = a.row_index[ci];
    const double lse_d = (double)mx + log((double)s);
    const float lse = (float)lse_d, logp = (float)((double)a.zt[ci] - lse_d);
    if (lane == 0) a.out_logp[slot] = logp;
    const float g = token_terms(a, slot, logp, q);
    if (write_dz) {
      const int y = a.targets[slot];
#pragma unroll
      for (int k = 0; k < LOGITS / 64; ++k) {
        const int v = k * 64 + lane;
        if (v < V) row[v] = g * ((v == y ? 1.f : 0.f) - expf(z[k] - lse));
      }
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < EPI_NQ; ++k) sh[wave][k] = q[k];
  }
  __syncthreads();
  if (threadIdx.x < EPI_NQ) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kRowWaves; ++w) t = threadIdx.x == 4 ? (sh[w][4] > t ? sh[w][4] : t) : t + sh[w][threadIdx.x];
    a.loss_partials[(a.partial_block_offset + blockIdx.x) * EPI_NQ + threadIdx.x] = t;
  }
}

constexpr int FIN_THREADS = 512;
__global__ __launch_bounds__(FIN_THREADS) void k_finalize(FinalizeArgs a) { finalize_block<FIN_THREADS>(a); }

// ----------------------------------------------------------------------------
// dz conversion of the fp32 path (proof of Prop. 4: grad log pi(a_i) = e_i - pi).
// ----------------------------------------------------------------------------
// fp32 path: scalar, bounds-checked.
__global__ __launch_bounds__(256) void k_convert_f32(float* ZP, int64_t ldz, const float* lse_c, const float* g_c,
                                                     const int32_t* targets, const int32_t* row_index,
                                                     const int64_t* n_scored, int64_t chunk_start,
                                                     int chunk_rows, int V) {
  const int nvalid = valid_rows(n_scored, chunk_start, chunk_rows);
  const int i = blockIdx.y;
  if (i >= nvalid) return;
  const int64_t ci = chunk_start + i;
  const float lse = lse_c[ci], g = g_c[ci];
  const int y = targets[row_index[ci]];
  for (int v = blockIdx.x * 256 + threadIdx.x; v < V; v += gridDim.x * 256) {
    const float p = expf(ZP[(int64_t)i * ldz + v] - lse);
    ZP[(int64_t)i * ldz + v] = g * ((v == y ? 1.f : 0.f) - p);
  }
}

// Backward operand of the dW launch, bf16: Ht[c][r] (or, in blocks of 32 rows, Ht[r / 32][c][r % 32]) = scale[r] * Hc[r][c] for the pass's valid
// rows, zeros up to the multiple of 128 the contraction runs over.  Tile 64 rows x 64 cols; n_cols a
// multiple of 64, 16-byte aligned rows on both sides.  The blocks behind the tiles clear the stash
// rows between the valid count and that multiple (the contraction must not meet stale bits there).
__global__ __launch_bounds__(256) void k_backward_rows_b16(const uint16_t* in, int64_t ld_in, const float* scale,
                                                           uint16_t* out, int64_t ld_out, const int64_t* n_scored,
                                                           int64_t chunk_start, int chunk_rows, int row_tiles,
                                                           uint16_t* E, int64_t lde, int Vp, bool in_blocks) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[64 * 72];
  const int nrows = valid_rows(n_scored, chunk_start, chunk_rows);
  const int nzero = (nrows + 127) / 128 * 128 < chunk_rows ? (nrows + 127) / 128 * 128 : chunk_rows;
  if ((int)blockIdx.y >= row_tiles) {
    const int i = nrows + blockIdx.y - row_tiles;
    if (i >= nzero) return;
    for (int v = (blockIdx.x * 256 + threadIdx.x) * 8; v < Vp; v += gridDim.x * 256 * 8)
      *reinterpret_cast<uint4*>(E + (int64_t)i * lde + v) = make_uint4(0, 0, 0, 0);
    return;
  }
  const int64_t r0 = (int64_t)blockIdx.y * 64;
  const int c0 = blockIdx.x * 64;
  if (r0 >= (nrows + 127) / 128 * 128) return;
  const int tc = threadIdx.x & 7, tr = threadIdx.x >> 3;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int rr = tr + 32 * k;
    const int64_t r = r0 + rr;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r < nrows) {
      const int c = c0 + tc * 8;
      v = *reinterpret_cast<const uint4*>(rows_in_blocks(chunk_rows) ? in + ((int64_t)(c / kRowBlock) * chunk_rows + r) * kRowBlock + c % kRowBlock
                                                                     : in + r * ld_in + c);
      // bf16 elements times the row's scale, rounded back to bf16 (nearest even)
      const float sc = scale[r];
      uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const __bf16 lo = (__bf16)(sc * bf16_bits_to_float(w[q] & 0xffffu));
        const __bf16 hi = (__bf16)(sc * bf16_bits_to_float(w[q] >> 16));
        uint16_t ul, uh;
        __builtin_memcpy(&ul, &lo, 2);
        __builtin_memcpy(&uh, &hi, 2);
        w[q] = (uint32_t)ul | ((uint32_t)uh << 16);
      }
      v = make_uint4(w[0], w[1], w[2], w[3]);
    }
    *reinterpret_cast<uint4*>(&tile[rr * 72 + tc * 8]) = v;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int cc = tr + 32 * k;
    uint32_t ow[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t lo = tile[(tc * 8 + q * 2) * 72 + cc];
      const uint32_t hi = tile[(tc * 8 + q * 2 + 1) * 72 + cc];
      ow[q] = lo | (hi << 16);
    }
    const int64_t r = r0 + tc * 8;
    uint16_t* const at = in_blocks ? out + ((r / kRowBlock) * (gridDim.x * 64) + c0 + cc) * kRowBlock + r % kRowBlock
                                   : out + (int64_t)(c0 + cc) * ld_out + r;
    *reinterpret_cast<uint4*>(at) = make_uint4(ow[0], ow[1], ow[2], ow[3]);
  }
}

}  // namespace

// ------------------------------------------------------------------ launchers
void launch_pad_rows_b16(const PadRows& p, hipStream_t stream) {
  hipLaunchKernelGGL(k_pad_rows_b16, dim3((unsigned)pad_blocks(p, 256)), dim3(256), 0, stream, p);
}

void launch_prep(const uint8_t* mask, const int32_t* targets, int64_t N, int V, const PrepOut& o, const PadRows& pad, hipStream_t stream) {
  const SlotOutputs zero = {{o.zero[0], o.zero[1], o.zero[2]}};
  const int64_t B = o.seq_len != nullptr ? o.B : 0;
  if (N <= kPrepOneBlock) {
    const int first_pad = (int)(1 + sequence_blocks(B, o.T, kPrepWaves));
    hipLaunchKernelGGL(k_prep_one, dim3((unsigned)(first_pad + pad_blocks(pad, kPrepThreads))), dim3(kPrepThreads), 0, stream,
                       mask, targets, (int)N, V, o.n_scored, o.n_bad, o.row_index, zero, B, o.T, o.seq_len, pad, first_pad);
    return;
  }
  if (pad.rows > 0) launch_pad_rows_b16(pad, stream);
  const int64_t nblocks = (N + PREP_PER_BLOCK - 1) / PREP_PER_BLOCK, seq_blocks = sequence_blocks(B, o.T, PREP_BLOCK / 64);
  // block_counts: [2 * nblocks] int32 counts followed (8-byte aligned) by [nblocks] int64 offsets
  int64_t* block_offsets = reinterpret_cast<int64_t*>(o.block_counts + round_up(2 * nblocks, 2));
  const bool scan = nblocks > kPrepMaxSelf;
  hipLaunchKernelGGL(k_prep_count, dim3((unsigned)(nblocks + seq_blocks)), dim3(PREP_BLOCK), 0, stream, mask, targets, N, V,
                     o.block_counts, nblocks, B, o.T, o.seq_len);
  if (scan)
    hipLaunchKernelGGL(k_prep_scan, dim3(1), dim3(1024), 0, stream, o.block_counts, nblocks, block_offsets,
                       o.n_scored, o.n_bad);
  hipLaunchKernelGGL(k_prep_fill, dim3((unsigned)nblocks), dim3(PREP_BLOCK), 0, stream, mask, targets, N, V,
                     o.block_counts, nblocks, scan ? block_offsets : nullptr, o.n_scored, o.n_bad, o.row_index, zero);
}

void launch_seq_log_ratio(const uint8_t* mask, const int32_t* targets, const float* logp,
                          const float* behav_logp, int64_t B, int T, int V, int level, float* seq_expo,
                          hipStream_t stream) {
  hipLaunchKernelGGL(k_seq_log_ratio, dim3((unsigned)B), dim3(256), 0, stream, mask, targets, logp, behav_logp,
                     T, V, level, seq_expo);
}

void launch_row_prep(RowPrepArgs a, int is_bf16, hipStream_t stream) {
  a.zero_blocks = a.dH != nullptr ? (a.N + ZERO_SLOTS_PER_BLOCK - 1) / ZERO_SLOTS_PER_BLOCK : 0;
  const int64_t blocks = (a.prep != nullptr ? 1 : 0) + (a.seq_coef != nullptr ? 1 : 0) + a.zero_blocks + (a.chunk_rows + 3) / 4;
  const PrepOut prep = a.prep != nullptr ? *a.prep : PrepOut{};
  auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, stream, a, prep); };
  if (a.prep != nullptr) { if (is_bf16) go(k_row_prep<true, true>); else go(k_row_prep<false, true>); }
  else if (is_bf16) go(k_row_prep<true, false>);
  else go(k_row_prep<false, false>);
}

void launch_row_lse_f32(const float* Z, int64_t ldz, const int64_t* n_scored, int64_t chunk_start,
                        int chunk_rows, int V, float* part_max, float* part_sum, float* part_ez,
                        hipStream_t stream) {
  hipLaunchKernelGGL(k_row_lse_f32, dim3(chunk_rows), dim3(256), 0, stream, Z, ldz, n_scored, chunk_start,
                     chunk_rows, V, part_max, part_sum, part_ez);
}

int row_epilogue_blocks(int chunk_rows) { return (chunk_rows + EPI_ROWS - 1) / EPI_ROWS; }

void launch_row_epilogue(const RowEpiArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(k_row_epilogue, dim3(row_epilogue_blocks(a.chunk_rows)), dim3(EPI_THREADS), 0, stream, a);
}

bool row_f32_fits(int V) { return V <= kRowLogits; }
int row_f32_blocks(int64_t rows) { return (int)((rows + kRowWaves - 1) / kRowWaves); }
void launch_row_f32(const RowEpiArgs& a, float* Z, int64_t ldz, int V, int rows, int write_dz, hipStream_t stream) {
  hipLaunchKernelGGL(V <= kFewLogits ? k_row_f32<kFewLogits> : k_row_f32<kRowLogits>, dim3(row_f32_blocks(rows)), dim3(kRowWaves * 64), 0, stream, a, Z, ldz, V, write_dz);
}

void launch_convert_f32(float* ZP, int64_t ldz, const float* lse_c,
                        const float* g_c, const int32_t* targets, const int32_t* row_index,
                        const int64_t* n_scored, int64_t chunk_start, int chunk_rows, int V,
                        hipStream_t stream) {
  int gx = (V + 255) / 256; gx = gx > 64 ? 64 : gx;
  dim3 grid(gx, chunk_rows);
  hipLaunchKernelGGL(k_convert_f32, grid, dim3(256), 0, stream, ZP, ldz, lse_c, g_c, targets,
                     row_index, n_scored, chunk_start, chunk_rows, V);
}

void launch_backward_rows_b16(const void* Hc, int64_t ldh, const float* scale, void* Ht, int64_t ldht,
                              const int64_t* n_scored, int64_t chunk_start, int chunk_rows, int dp, void* E, int64_t lde,
                              int Vp, bool in_blocks, hipStream_t stream) {
  const int row_tiles = chunk_rows / 64;
  hipLaunchKernelGGL(k_backward_rows_b16, dim3(dp / 64, (unsigned)(row_tiles + 127)), dim3(256), 0, stream,
                     static_cast<const uint16_t*>(Hc), ldh, scale, static_cast<uint16_t*>(Ht), ldht, n_scored,
                     chunk_start, chunk_rows, row_tiles, static_cast<uint16_t*>(E), lde, Vp, in_blocks);
}

void launch_finalize(const FinalizeArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(k_finalize, dim3(1), dim3(FIN_THREADS), 0, stream, a);
}

}  // namespace mrl
