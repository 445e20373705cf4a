/*
 * mrl_diag.h - measurement aids of the MI355X GRPO scoring library.
 *
 * Not part of the product boundary (include/mrl.h): a training or serving loop needs none of
 * this.  The benchmark uses these calls to time the kernel classes of a step with HIP events
 * on the launch stream (the figures behind its roofline object) and to measure what the matrix
 * cores of the box sustain with no memory traffic.  Same conventions as mrl.h: mrl_status
 * return codes, device pointers owned by the caller, nothing allocated on the device.
 */
#ifndef MRL_DIAG_H
#define MRL_DIAG_H

#include <stddef.h>
#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* ------------------------------------------------------------------------
 * Per-kernel-class timing for benchmarks.  When enabled, every kernel launch
 * of the entry points of mrl.h is bracketed by HIP events on the launch stream.
 * mrl_profile_collect synchronises the device, adds up the elapsed time and
 * launch count per class since the last collect, and resets the log.
 * Arrays are HOST memory of MRL_PROF_NCLASS entries.
 * ---------------------------------------------------------------------- */
enum {
  MRL_PROF_PREP = 0,      /* mask scan, compaction, scored lengths, zeros of unscored slots' outputs but dH (calls of more than 2048 slots), padded copy of W's columns */
  MRL_PROF_ADV = 1,       /* group advantages */
  MRL_PROF_GEMM_FWD = 2,  /* logits tile GEMM with fused log-sum-exp */
  MRL_PROF_ROW_EPI = 3,   /* partial merge, ratio / clip / KL, loss partials (fp32 loss calls of at most 2048 ids: log-sum-exp and logits -> dz as well, one launch) */
  MRL_PROF_CONVERT = 4,   /* operand preparation: row gather and target logits, sequence weights, zero dH rows, and up to 2048 slots what PREP does with the mask above; scaled transpose (fp32 loss calls of more ids: logits -> dz) */
  MRL_PROF_GEMM_DH = 5,   /* dH = dz W; fp32 passes too small to fill the chip with either product: both, and in the last pass the final reductions, as the one launch they are */
  MRL_PROF_GEMM_DW = 6,   /* dW += dz^T H (nothing for those fp32 passes) */
  MRL_PROF_FINAL = 7,     /* final reductions (nothing where they came with that launch) */
  MRL_PROF_NCLASS = 8
};
int mrl_profile_enable(int on);
int mrl_profile_collect(double* ms_per_class /*host*/, int64_t* launches_per_class /*host*/);

/* ------------------------------------------------------------------------
 * Diagnostic: sustained rate of the matrix cores on the MFMA instruction the
 * GEMM kernels use (bf16 16x16x32, fp32 accumulate), registers only, no memory
 * traffic.  random_operands = 0: constant operands (clock-limited peak);
 * 1: random sign / mantissa operands, which is what activations and weights
 * look like - the device lowers its clock under the higher switching power, so
 * this is the ceiling of any bf16 GEMM on real data.  Benchmarks print both
 * next to the published peak (Sec. 3 defines the contraction this bounds).
 * Synchronous: runs on the null stream for about `seconds` (0 < seconds <= 5)
 * and waits.  scratch: device memory, at least 1024 bytes per compute unit
 * (512 KiB is enough for any device); out_tflops: host.  Errors: MRL_ERR_NULL,
 * MRL_ERR_CONFIG (seconds), MRL_ERR_WORKSPACE (scratch too small), MRL_ERR_DEVICE.
 * ---------------------------------------------------------------------- */
int mrl_probe_mfma_rate(int32_t random_operands, double seconds, void* scratch /*dev*/,
                        size_t scratch_bytes, double* out_tflops /*host*/);

/* ------------------------------------------------------------------------
 * The launch plan of the dW GEMM for an LM head of V rows and d columns where
 * it runs on 256 x 256 tiles (short contractions; mrl_diag_gemm_cut says which) (host code only, no GPU call): which rows of 256 x 256 tiles are cut into slices of
 * the contraction at the end of the launch, into how many, and how many of the
 * resulting work items each of the 8 XCDs takes.  For tests of the host logic
 * and for reading profiles.  out12 (host): [0] first tile row of the tail,
 * [1] tile rows in the tail, [2] slices per tile (0: the tiles stay whole),
 * [3 + x], x = 0..8: items before XCD x (so [11] is the item count).
 * Errors: MRL_ERR_NULL, MRL_ERR_SHAPE (V or d not positive).
 * ---------------------------------------------------------------------- */
int mrl_diag_dw_tail_plan(int32_t V, int32_t d, int32_t* out12 /*host*/);

/* ------------------------------------------------------------------------
 * Rows up to which a pass of the bf16 loss takes the dW launch for few rows, which has
 * no tail (host code only): as many as the pass can hold, or as scored_rows_hint says
 * that it will.  For tests that mean to run the one launch or the other.
 * ---------------------------------------------------------------------- */
int mrl_diag_dw_few_rows(void);

/* ------------------------------------------------------------------------
 * The slices of the contraction that each of the tail_tiles (1 .. 255) tiles of
 * the dH launch's last, incomplete round of 256 is cut into (1: left whole), for
 * a contraction of `panels` panels of 64 and scratch for max_items partial tiles:
 * the function that the launch and its reduction evaluate on the device (host
 * code here, no GPU call).  Errors: MRL_ERR_SHAPE.
 * ---------------------------------------------------------------------- */
int mrl_diag_dh_split(int32_t tail_tiles, int32_t panels, int32_t max_items);

/* ------------------------------------------------------------------------
 * The tiles of a large bf16 launch (host code only, no GPU call), for tests that mean to reach one
 * path or the other.  launch: MRL_PROF_GEMM_FWD, _DH or _DW; rows: valid rows of the pass (FWD: of the launch's part of it);
 * expected (DW): rows at most, as far as scored_rows_hint says, else chunk_rows; chunk_rows: length of the pass (or
 * part), a multiple of 256; tail_items: partial tiles the workspace has room for (0: the full size's).
 * out9 (host): [0] tiles of 384, [1] of 256, [2] of 128 along the token rows (DW: the vocabulary), [3] tiles of the launch, [4] those
 * of its last round, which may be cut, [5] slices of the contraction that each of them is cut into (1: whole), [6] workgroups launched (DW on
 * 256 x 256 tiles: for the whole tiles), [7] tail_items, [8] first row of the last tile along the token rows.  FWD of passes of at most 256
 * rows and DW of at most mrl_diag_dw_few_rows() have launches of their own (DW: all zeros but [7]).  Errors: MRL_ERR_NULL, MRL_ERR_SHAPE.
 * ---------------------------------------------------------------------- */
int mrl_diag_gemm_cut(int32_t launch, int32_t rows, int32_t expected, int32_t chunk_rows, int32_t V, int32_t d, int32_t tail_items,
                      int32_t* out9 /*host*/);

#ifdef __cplusplus
}
#endif
#endif /* MRL_DIAG_H */
