// Internal declarations shared by the library's translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace mrl {

// Column padding of the per-chunk logit / dz buffers: the vocabulary is padded
// to a multiple of the GEMM tile so that inner kernels never see a ragged K.
constexpr int kTile = 256;
inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// A kernel that asks for more than 64 KB of dynamic LDS needs its limit raised first; the
// attribute belongs to the (kernel, device) pair, so it is set once on every device used.
struct LdsLimit {
  std::atomic<bool> done[64] = {};
  void ensure(const void* kernel, int bytes) {
    int dev = 0;
    (void)hipGetDevice(&dev);
    const bool tracked = dev >= 0 && dev < 64;
    if (tracked && done[dev].load(std::memory_order_acquire)) return;
    (void)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (tracked) done[dev].store(true, std::memory_order_release);
  }
};

// Passes of at most kFewRows rows hold the gathered rows in blocks of kRowBlock columns, [dp / 32][chunk_rows][32],
// instead of row by row: what the forward kernel of such passes loads at a time is then contiguous.  (The last part
// of a longer pass may have as few rows; it runs on the large tile like the other parts.)
constexpr int kFewRows = 256, kRowBlock = 32;
__host__ __device__ inline bool rows_in_blocks(int chunk_rows) { return chunk_rows <= kFewRows; }

// Number of sum-exp partials each token row receives from the forward kernel: the bf16
// kernel emits two per 256-wide vocabulary tile (one per wave row), the fp32 path a single
// (max, sum-exp) pair per row.
inline int fwd_partials_bf16(int V) { return 2 * (int)((V + kTile - 1) / kTile); }

// bf16 path: exponentials are taken relative to a per-row offset that is known before the forward
// launch, c2[n] = z_t[n] * log2(e) + kStashMargin2 (log2 domain, z_t = the row's target logit):
//   e[n, v] = 2^(min(z[n, v] * log2(e) - c2[n], kStashClamp2)),   S[n] = sum_v e[n, v].
// One offset for the whole row is what lets the forward kernel write e itself (as bf16) for the
// backward pass: softmax = e / S, so dz = g (onehot - e / S) = (-g / S) (e - S onehot) is the
// stored row, patched at the target column, times a per-row scalar that the dH epilogue applies
// to its output rows and that the dW launch finds folded into its copy of the hidden rows.
// Relative to the target logit nothing of weight can underflow (e >= p * 2^-margin) and the
// largest entry is exp(-logp_target) * 2^-margin.  With margin 60 and clamp 100 every quantity
// stays a normal bf16 / fp32 number for log-probs of the target down to about -97; below that
// the row saturates (finite, inexact) and is counted.
constexpr float kStashMargin2 = 60.f;
constexpr float kStashClamp2 = 100.f;
constexpr float kSaturatedLogp = -97.f;

// ---- bf16 MFMA GEMM family: C[m][n] = sum_k A[m][k] * B[n][k] ---------------
// n_scored: device pointer to the number of compacted rows; chunk_start/chunk_rows
// select the rows this launch covers (valid rows = clamp(n_scored - chunk_start, 0, chunk_rows)).

// Forward: A = W [V, k_len] (row stride ldw), B = Hc [chunk_rows, k_len] (row stride ldh, or, in_blocks, in
// blocks of kRowBlock columns of ldh rows each): the launch's token rows, gathered; k_len = d rounded up to 128, the columns beyond d
// zero in both operands; zt[chunk_start + n] is the row's target logit.  Writes per-row partials part_sum[(2*tile_m + wave_m) * part_stride + n]
// = sum of e[n, v] over the partial's 128 vocabulary rows (e as defined above), when part_ez != nullptr
// also sum e * z (for the entropy), and, when estash != nullptr, e itself as bf16 into
// estash[n * lde + v] (n = row within this launch; columns V .. round_up(V, 256) get zeros).
// W_tail (nullptr: none): the last 128 columns of the K extent, zero-padded, in rows of the same stride
// ldw; the other columns are read from W, whose rows need not reach that far.
void launch_gemm_fwd_bf16(const void* W, int64_t ldw, const void* W_tail, const void* Hc, int64_t ldh, int k_len, const float* zt,
                          const int64_t* n_scored, int64_t chunk_start, int chunk_rows,
                          int V, int d, float* part_sum, float* part_ez,
                          int64_t part_stride, void* estash, int64_t lde, bool in_blocks, hipStream_t stream);

// dH: A = E [chunk_rows, Vp] (the patched bf16 stash), B = W^T read in place from W [V, d] (row
// stride ldw); row m, multiplied by row_scale[chunk_start + m], goes to
// dH[row_index[chunk_start + m], :] as bf16 (dh_f32 = 0) or float (dh_f32 = 1).
// tail_part: scratch of tail_items * gemm_tail_tile_bytes() bytes for the K slices of the last
// round's tiles.
void launch_gemm_dh_bf16(const void* E, int64_t lde, const void* W, int64_t ldw, int V,
                         const int32_t* row_index, const float* row_scale, const int64_t* n_scored,
                         int64_t chunk_start, int chunk_rows, int d, void* dH, int dh_f32,
                         float* tail_part, int tail_items, hipStream_t stream);

// dW: A = E^T read in place from E [chunk_rows, Vp] (rows >= valid rows rounded up to 128 and
// columns >= V must be zero), B = Ht [d, chunk_rows] (the pass's hidden rows, each already
// multiplied by its row scale); dW[v, :] = (or +=) sum over the chunk's valid rows.
// overwrite = 1 stores, 0 adds into the existing values.
// tail_part: scratch of tail_items * gemm_tail_tile_bytes() bytes (gemm_tail_bytes_least() or more) for the K slices of the last
// tiles; rows: the scored rows expected (which tiles the launch takes; right for any number).
// in_blocks: the launch for few rows, with Ht in blocks of kRowBlock token rows, [chunk_rows / 32][ldht][32], ldht = d
// rounded up to 128; dw_rows_in_blocks says where it is the faster one (rows: the scored rows expected; right for any number).
size_t gemm_tail_tile_bytes();
int gemm_tail_items(size_t head_bytes);               // of a workspace, for a head of so many bytes
size_t gemm_tail_bytes_least(size_t head_bytes);      // ... in one that has no room for them all
bool dw_rows_in_blocks(int rows);
void launch_gemm_dw_bf16(const void* P, int64_t ldp, const void* Ht, int64_t ldht,
                         const int64_t* n_scored, int64_t chunk_start, int chunk_rows,
                         int V, int d, float* dW, int overwrite, float* tail_part, int tail_items, int rows, bool in_blocks,
                         hipStream_t stream);

// ---- fp32 GEMM (small-shape path): C[m][n] = sum_k A[m][k] * B[n][k] --------
// An operand is k-contiguous (element (row, k) at row * ld + k) or, with its kmajor flag, stored with
// k as the row (at k * ld + row).  a_rows / b_rows: optional maps of the operand's stored rows, c_rows
// of the output's (index arrays already offset to the chunk).  Supported: neither k-major, B, both.
// M is computed on the device from n_scored when m_dynamic != 0, K likewise when k_dynamic != 0.
struct GemmF32Args {
  const float* A; int64_t lda; const int32_t* a_rows; int a_kmajor;
  const float* B; int64_t ldb; const int32_t* b_rows; int b_kmajor;
  float* C; int64_t ldc; const int32_t* c_rows;
  int M, N, K;
  const int64_t* n_scored; int64_t chunk_start; int chunk_rows;
  int m_dynamic, k_dynamic;
  int accumulate;
  int m_on_x;   // set by the launcher
};
void launch_gemm_f32(const GemmF32Args& a, hipStream_t stream);
// Both products in one launch (a: B k-major; b: both k-major), where gemm_f32_pairs says that neither
// fills the chip.
// `last`, if not nullptr: the call's last launch, and the statistics come with it.
struct FinalizeArgs;
bool gemm_f32_pairs(const GemmF32Args& a, const GemmF32Args& b);
void launch_gemm_f32_pair(const GemmF32Args& a, const GemmF32Args& b, const FinalizeArgs* last, hipStream_t stream);

// ---- auxiliary kernels ------------------------------------------------------
struct PrepOut {
  int32_t* row_index;   // [N] compacted scored slots, in slot order; tail filled with 0
  int64_t* n_scored;    // [1]
  int64_t* n_bad;       // [1] masked-in slots with a target outside [0, V)
  int32_t* block_counts; // scratch: per 1024-slot block a scored count and a bad-target count (int32),
                         // followed, 8-byte aligned, by the blocks' exclusive offsets (int64)
  float* zero[3];       // per-slot outputs that unscored slots set to 0 (or nullptr)
  int64_t B; int T; int32_t* seq_len;   // scored slots (valid targets only) per sequence of T slots, if not nullptr
};
// out[r][0:dp] = in[r][0:d], zero in [d, dp), r < rows (0: nothing to do).  16-byte vectors: d, dp, both row strides
// multiples of 8 elements, both pointers 16-byte aligned.
struct PadRows { const void* in; int64_t ld_in; void* out; int64_t ld_out; int64_t rows; int d, dp; };
void launch_pad_rows_b16(const PadRows& p, hipStream_t stream);
// The compaction, and what of W is to be padded.
void launch_prep(const uint8_t* mask, const int32_t* targets, int64_t N, int V, const PrepOut& o, const PadRows& pad,
                 hipStream_t stream);
// Calls of at most kPrepInline slots take no launch_prep: the first launch_row_prep of the call is given its outputs.
// (Every block scans all slots, in a loop unrolled to this length.  Scoring calls, d = 64, V = 1000, us, with a launch and inline: 201
// slots 22.3 and 19.1, 1024 25.4 and 22.9, 2048 26.2 and 23.8.  Unrolled to 4096 it takes 24.9 at 2048 slots, 26.0 at 3003
// and 27.2 at 4096 against 26.5 and 27.1 with a launch: what the longer loop gives there it costs the smaller calls.)
constexpr int64_t kPrepInline = 2048;
inline bool prep_inline(int64_t N) { return N <= kPrepInline; }

// Response-level log-ratio (App. I.1): seq_expo[b] = sum over the scored tokens of sequence b of
// (logp - behav_logp), divided by the number of scored tokens when level == 2.  Fixed-order
// reduction, one workgroup per sequence.
void launch_seq_log_ratio(const uint8_t* mask, const int32_t* targets, const float* logp,
                          const float* behav_logp, int64_t B, int T, int V, int level, float* seq_expo,
                          hipStream_t stream);

// Before a pass's forward launch: target logit z_t[i] = <H[row_index[i]], W[target]> of its rows (fp32
// accumulate) and, on the bf16 path, their copies Hc[r][0:dp] = H[row][0:d] | 0 (16-byte vectors: d,
// dp, ldh multiples of 8).  With the first pass of a loss call also the zero dH rows of unscored
// slots (dH != nullptr) and the sequence weights (seq_coef != nullptr): seq_coef[b] = 1 / (P K_g L_b)
// for GRPO rows, 1 / (S_aux L_b) for SGT rows, 0 for empty rows.
struct RowPrepArgs {
  const void* H; const void* W; const int32_t* targets; const int32_t* row_index; const int64_t* n_scored;
  int64_t chunk_start; int chunk_rows; int d;
  void* Hc; int64_t ldh; int dp;   // (in blocks of kRowBlock columns, chunk_rows rows each, where rows_in_blocks says so)
  float* zt;
  const uint8_t* mask; int64_t N; int V; void* dH; int64_t dh_row_bytes; int64_t zero_blocks /*set by the launcher*/;
  const int32_t* seq_len; const int32_t* group_id; const uint8_t* seq_kind; int64_t B; int G; int loss_agg;
  int32_t* group_count /*[G] scratch*/; float* seq_coef;
  int64_t* n_bad_groups /*[1]: sequences whose group id is outside [0, G)*/;
  const PrepOut* prep;             // not nullptr: mask and targets are compacted here, too (prep_inline; mask, N, V are set)
};
void launch_row_prep(RowPrepArgs a, int is_bf16, hipStream_t stream);

// fp32 path: (max, sum-exp[, sum exp * z]) of each row of Z [rows, V] -> one partial per row.
void launch_row_lse_f32(const float* Z, int64_t ldz, const int64_t* n_scored, int64_t chunk_start,
                        int chunk_rows, int V, float* part_max, float* part_sum, float* part_ez,
                        hipStream_t stream);

struct RowEpiArgs {
  // part_max == nullptr: part_sum holds the bf16 kernel's offset sums (see kStashMargin2);
  // else (fp32 path) one (max, sum exp(z - max)) pair per row
  const float* part_max; const float* part_sum; int n_partials; int chunk_rows;
  const float* part_ez; float* out_entropy;   // both nullptr unless the entropy is asked for (per slot)
  const float* zt;            // [N] compacted
  const int32_t* row_index; const int64_t* n_scored; int64_t chunk_start;
  // loss inputs (all nullptr for the log-prob-only entry point)
  const float* behav_logp; const float* ref_logp; const float* seq_adv;
  const float* seq_coef; const uint8_t* seq_kind; int T;
  // response-level ratio (App. I.1): exponent per sequence, lengths, level 1 (sum) or 2 (mean); null = token ratio
  const float* seq_expo; const int32_t* seq_len; int ratio_level;
  float eps_lo, eps_hi, beta, lambda;
  float* out_logp; float* out_lse;  // per slot
  float* lse_c; float* g_c;         // per compacted row (nullptr to skip)
  // bf16 backward: row_scale[ci] = -g / S, and the stash row's target column becomes e - S
  float* row_scale; uint16_t* estash; int64_t lde; const int32_t* targets;
  double* loss_partials;            // [n_blocks_total][8], block index = chunk block offset + blockIdx
  int64_t partial_block_offset;
};
int row_epilogue_blocks(int chunk_rows);
void launch_row_epilogue(const RowEpiArgs& a, hipStream_t stream);

// fp32 path, V small enough (row_f32_fits): log-sum-exp of the materialised logits, row epilogue and, with write_dz, conversion
// to dz in one launch.  Of a: part_max .. out_entropy, lse_c, g_c and row_scale are not used; a loss partial per
// row_f32_blocks' block of rows.  rows: those the pass can have (at most chunk_rows).
bool row_f32_fits(int V);
int row_f32_blocks(int64_t rows);
void launch_row_f32(const RowEpiArgs& a, float* Z, int64_t ldz, int V, int rows, int write_dz, hipStream_t stream);

// fp32 path, dz conversion: P[i][v] = g_i (1[v = y_i] - exp(z - lse_i)) in place of the chunk's logits.
void launch_convert_f32(float* ZP, int64_t ldz, const float* lse_c,
                        const float* g_c, const int32_t* targets, const int32_t* row_index,
                        const int64_t* n_scored, int64_t chunk_start, int chunk_rows, int V,
                        hipStream_t stream);

// bf16 path, operands of the dW launch (Hc as the row preparation wrote it): Ht[c][r] = scale[r] * Hc[r][c] (c < dp, a multiple of 64) for the
// pass's valid rows, zeros up to their multiple of 128; the stash rows in between are cleared (the
// dW contraction runs over pairs of 64-row panels; the forward kernel writes valid rows only).
// in_blocks: Ht[r / 32][c][r % 32] instead.
void launch_backward_rows_b16(const void* Hc, int64_t ldh, const float* scale, void* Ht, int64_t ldht,
                              const int64_t* n_scored, int64_t chunk_start, int chunk_rows, int dp, void* E, int64_t lde,
                              int Vp, bool in_blocks, hipStream_t stream);

// Group-relative advantages (Sec. 3) with pooled / own statistics and SGT gate flags.
void launch_group_advantages(const float* rewards, const int32_t* group_id, const uint8_t* in_stats,
                             const uint8_t* scored, const uint8_t* is_own, const float* baseline_shift,
                             int64_t B, int G, int mode, float eps_norm, int ddof, float mix_alpha, float neg_thresh,
                             float pos_thresh, float* out_adv, float* out_mean, float* out_std,
                             uint8_t* out_flags, hipStream_t stream);

// End of a loss call.  rows_enqueued: number of compacted rows covered by the enqueued passes; scored rows beyond
// it (a wrong scored_rows_hint) get NaN log-probs and are counted in the stats.
struct FinalizeArgs {
  const double* parts; int64_t n_blocks; const int64_t* n_scored; const int64_t* n_bad; float beta, lambda;
  int64_t rows_enqueued; const int32_t* row_index; float* out_logp; double* out_d; int64_t* out_i;
};
void launch_finalize(const FinalizeArgs& a, hipStream_t stream);

// MRL_OK when the current device is a gfx950, else MRL_ERR_UNSUPPORTED_ARCH / MRL_ERR_DEVICE.
int require_gfx950();

// ---- profiling ---------------------------------------------------------------
void prof_begin(int cls, hipStream_t stream);
void prof_end(int cls, hipStream_t stream);

}  // namespace mrl
