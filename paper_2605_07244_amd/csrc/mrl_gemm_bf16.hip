// bf16 MFMA tile GEMM for gfx950 with three fused epilogues.
//
// One kernel body computes C[m][n] = sum_k A[m][k] * B[n][k] for a 256 x 256
// tile per workgroup (both operands K-contiguous, "NT" form).  Four wave64
// wavefronts form a 2 x 2 grid, each owning a 128 x 128 sub-tile as 8 x 8
// MFMA 16x16x32 accumulators (256 accumulator registers per lane).  The
// 16x16x32 shape is chosen over 32x32x16 for energy: with real (random-mantissa)
// operands the chip is power-limited, and an MFMA-only loop sustains about 13 %
// more FLOP/s with the 16 x 16 shape.  Operand panels of 64 K-elements go from
// global memory straight into LDS (global_load ... lds, no staging registers)
// into a double buffer.  LDS rows are 128 bytes whose 16-byte chunks are
// XOR-swizzled with (row / 2) % 8: a 128-bit LDS read is served 16 lanes (16
// rows of one chunk column) per cycle over 64 banks, rows 2 apart share a bank
// window, and the swizzle spreads them over the eight chunk slots, so the
// fragment reads of the MFMA operands are bank-conflict free; the swizzle is
// applied on the global side (each lane picks the chunk whose LDS slot it owns)
// because a direct load writes the wave's 64 x 16 bytes contiguously.
//
// The three uses on the scoring path (Sec. 3: log pi(y_t | ...) needs the
// softmax over the whole vocabulary of the LM-head logits):
//   FWD: A = W (vocabulary rows), B = H (token rows, gathered).  The MFMA result
//        layout keeps 4 rows x 1 column per lane, so putting the vocabulary on
//        the M side makes the max / sum-exp reduction over the vocabulary an
//        in-register reduction with two cross-lane steps.  The fragment rows are
//        permuted so that a lane's accumulators are 8 consecutive vocabulary ids
//        and the stash of exponentials e = exp(z - row offset) is stored as bf16
//        straight from registers.
//   DH : A = stash rows (tokens), B = W^T, read from the rows of W themselves (K-major
//        panel, transposing LDS reads); each output row is multiplied by its row scale
//        (-g / S) and scattered to its slot.
//   DW : A = stash^T, read from the stash rows themselves (K-major panel, transposing
//        LDS reads), B = (row-scaled H)^T; fp32 read-modify-write of dW.
#include "../../include/mrl.h"
#include "../../include/mrl_diag.h"
#include "mrl_internal.h"

namespace mrl {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte access, 4-byte alignment

constexpr int BM = 256, BN = 256, BK = 64;
constexpr int NTHREADS = 256;
constexpr int NSTAGE = 2;                          // LDS double buffer of K panels
constexpr int TILE_BYTES = BM * BK * 2;            // one operand panel: 32 KB (256 rows x 128 B)
constexpr int STAGE_BYTES = 2 * TILE_BYTES;        // A + B
constexpr int DHSTAGE_LD = BM + 8;                   // bf16 elements per row of the dH epilogue's staging tile
constexpr int DHSTAGE_BYTES = BN * DHSTAGE_LD * 2;     // 132 KB
constexpr int PIPE_BYTES = NSTAGE * STAGE_BYTES;   // 128 KB
// Direct loads of a slot's 16 (per wave), by the group of the K loop that issues them: the slot is
// released by the barrier in group 5, so its refill starts there and may run on into groups 0 - 4
// of the next panel (it is needed at that panel's barrier).
constexpr int kLoadsInGroup[8] = {4, 0, 0, 0, 0, 4, 4, 4};
constexpr int load_index_base(int g) {      // loads issued before group g, in the order 5, 6, 7, 0, 1, ...
  int n = 0;
  for (int h = 5; h != g; h = (h + 1) & 7) n += kLoadsInGroup[h];
  return n;
}
constexpr int kLoadsCarriedOver = kLoadsInGroup[0] + kLoadsInGroup[1] + kLoadsInGroup[2] + kLoadsInGroup[3] + kLoadsInGroup[4];
static_assert(kLoadsCarriedOver + kLoadsInGroup[5] + kLoadsInGroup[6] + kLoadsInGroup[7] == 16, "a slot takes 16 loads per wave");
constexpr int kDwTailMaxItems = 256;                // K slices of dW tail tiles per launch: one per compute unit
constexpr int ZT_BYTES = BN * 4;                   // forward: the tile's 256 target logits, behind the panels
template <int MODE> constexpr int lds_bytes() {     // (forward: the half-column tiles keep three stages of 48 KB)
  return MODE == 0 ? PIPE_BYTES + TILE_BYTES / 2 + ZT_BYTES : (DHSTAGE_BYTES > PIPE_BYTES ? DHSTAGE_BYTES : PIPE_BYTES);
}

// s_waitcnt immediates (gfx9 encoding): wait until at most N vector-memory loads are
// outstanding, no wait on the export / LDS counters.
constexpr int waitcnt_vm(int n) { return (n & 0xF) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }

enum { MODE_FWD = 0, MODE_DH = 1, MODE_DW = 2 };
constexpr int NXCD = 8;
template <bool B> struct Flag { static constexpr bool value = B; };

struct Params {
  const uint16_t* A; int64_t lda; int M;
  const uint16_t* B; int64_t ldb; int N;
  int K;
  const int32_t* row_index;   // already offset to the chunk start
  const int64_t* n_scored; int64_t chunk_start; int chunk_rows;
  int sup_m, sup_n;           // DW: super-tile shape of the workgroup -> tile mapping
  // FWD; a_tail_panel: the 64-wide panel from which A comes from its zero-padded tail copy, a_tail_delta
  // bytes behind where it would be
  int a_tail_panel; int64_t a_tail_delta;
  const float* zt; float* part_sum; float* part_ez; int64_t part_stride; uint16_t* estash; int64_t lde; int V;
  // DH
  const float* row_scale; void* dH; int dh_f32; int d; int max_items;   // max_items: partial tiles tail_part holds
  // DW
  float* dW; int overwrite; int streaming;
  // DW, K-split tail (see dw_tail_plan): workgroups from main_blocks on take the tiles of the
  // tile rows tail_m0 .. tail_m0 + tail_rows - 1, each cut into tail_split slices of the
  // contraction, and store their accumulators to tail_part instead of dW
  int main_blocks, tail_m0, tail_rows, tail_split; float* tail_part;
  int tail_first[NXCD + 1];   // items tail_first[x] .. tail_first[x + 1] - 1 run on XCD x
};

// Workgroup -> tile mapping of the forward and dH launches.  Workgroups are dealt round-robin to the
// 8 XCDs, each with its own L2 and 32 compute units; 32 consecutive workgroups of one XCD take 32
// consecutive tiles, numbered down the columns of bands of 8 tile rows (8 x 4 tiles when the N extent
// allows), so that they share operand panels in that L2 and all XCDs walk the same A rows at the same
// time.  The numbering runs over the VALID tiles (the scored rows are counted on the device) without
// holes: numbering super-tiles over the launch's upper bound gave each XCD fixed tile columns, and
// with 20 of 32 tile columns valid three XCDs had nothing to do (scoring 5120 of 8192 slots,
// V = 128256, d = 2048: 3233 us a call against 2088 us now).  The tiles of the last, incomplete round
// of 256 are dealt evenly.
constexpr int kBand = 8;
constexpr int kXcdCus = 32;
constexpr int kRound = NXCD * kXcdCus;
__device__ inline void tile_at(int t, int Mt, int Nt, int& tm, int& tn) {
  const int band = t / (kBand * Nt), in_band = t - band * kBand * Nt;
  const int rows = Mt - band * kBand < kBand ? Mt - band * kBand : kBand;
  tn = in_band / rows;
  tm = band * kBand + in_band - tn * rows;
}
__device__ inline bool dealt_tile(int bid, int Mt, int Nt, int& tm, int& tn) {
  const int tiles = Mt * Nt, whole = tiles / kRound * kRound;
  const int xcd = bid % NXCD, local = bid / NXCD;
  int t;
  if (bid < whole) {
    t = (local / kXcdCus * NXCD + xcd) * kXcdCus + local % kXcdCus;
  } else {
    const int per = (tiles - whole + NXCD - 1) / NXCD, k = local - whole / NXCD;
    t = whole + xcd * per + k;
    if (k >= per || t >= tiles) return false;
  }
  tile_at(t, Mt, Nt, tm, tn);
  return true;
}

// dH: the tiles of the last, incomplete round of 256 (all of them, when a pass has few rows) are cut
// into slices of the contraction over the vocabulary, one work item each, which store their
// accumulators to a scratch area; dh_tail_reduce adds them in slice order.  A dH tile is long (2374
// panels at V = 151936, about 2.4 ms), so an idle compute unit in that round costs more than
// writing and adding the partial tiles (256 KB per item): 327 rows at d = 4096 are 32 tiles.
// The slice count is the one whose rounds of items end earliest, 1 / kItemCostInv of a tile covering an item's
// prologue, partial store and share of the reduce.  In whole numbers: the launch and the reduction each work
// it out on the device and have to come to the same answer.  Measured (launch and reduce, V = 151936; before:
// whole tiles and a transposed copy of W in front): 327 rows, d = 4096, 32 tiles: 3480 -> 527 us;
// 5120 rows, d = 1536, 120 tiles: 3251 -> 1720 us; 47360 rows, d = 3584, 2590 tiles: 39.1 -> 35.9 ms.
constexpr int kMinSlicePanels = 16;
__host__ __device__ inline int dh_split(int tail_tiles, int panels, int max_items) {
  constexpr int kItemCostInv = 50;
  int best = 1, best_num = 1, best_den = 1;        // when the last item ends, in tiles: rounds * (1 / s + 1 / kItemCostInv)
  for (int s = 2; s <= 64 && s * kMinSlicePanels <= panels && s * tail_tiles <= max_items; ++s) {
    const int rounds = (tail_tiles * s + kRound - 1) / kRound;
    const int num = rounds * (kItemCostInv + s), den = kItemCostInv * s;   // (cross products below 2^25)
    if (num * best_den < best_num * den) { best_num = num; best_den = den; best = s; }
  }
  return best;
}
// Work items of the last round at most, whatever the scored rows.  Launching what the scratch holds instead made
// passes without rows slower than before the slices (47 passes of 1024 rows, 3 with rows, V = 705, d = 3040, no hint:
// 1800 us a call before, 1750 - 1911 with them, now 1640), and below 32 panels (V <= 1920) nothing is
// sliced and the reduction is left out.
inline int dh_most_split(int panels) { return panels / kMinSlicePanels < 2 ? 1 : (panels / kMinSlicePanels < 64 ? panels / kMinSlicePanels : 64); }
inline int dh_most_items(int tiles, int panels, int max_items) {
  const int n = (tiles < kRound ? tiles : kRound - 1) * dh_most_split(panels);
  return n < max_items ? n : max_items;
}
// panels per slice: an even number (the K loop's body is two panels)
__host__ __device__ inline int slice_panels(int panels, int split) { return ((panels + split - 1) / split + 1) & ~1; }
// slices that have any panels: the dW plan does not know the scored rows, and 6 panels make three slices of the
// planned 8.  (No panels at all: the first slice stores the zeros of an overwriting launch.)
__device__ inline int slices_in_use(int panels, int split) {
  const int per = slice_panels(panels, split);
  return panels > 0 ? (panels + per - 1) / per : 1;
}
// panels of the dW contraction: the pass's valid rows, rounded up to panel pairs
__device__ inline int dw_panels(int nvalid, int chunk_rows) {
  const int k = (nvalid + 2 * BK - 1) / (2 * BK) * (2 * BK);
  return (k < chunk_rows ? k : chunk_rows) / BK;
}

// Workgroup -> tile mapping of the dW launch (its tile counts do not depend on the scored rows):
// sup_m x sup_n consecutive workgroups of one XCD form a super-tile (each A panel is used by sup_n
// tiles, each B panel by sup_m), and super-tiles are numbered N-fastest so that the XCDs walk the
// same A rows at the same time.  The shape is picked per launch from what measurement favours: 8 x 4
// when the N extent is a multiple of 4 tiles, else 8 x 2.  Two things matter more than the
// panel-sharing count: the N extent must fill whole super-tile columns (6 tiles at d = 1536 and 14 at
// d = 3584 leave 8 x 4 with a half-empty last column: 11-30 % slower than 8 x 2), and the super-tile
// size must divide the 32 compute units of an XCD, so that the workgroups running on it at any time
// are whole super-tiles (shapes of 24, 28 or 30 tiles lose 5-20 %).
struct SuperTile { int m, n; };
inline SuperTile pick_super_tile(int Nt) {
  if (Nt % 4 == 0) return {8, 4};
  if (Nt == 1) return {16, 1};
  return {8, 2};
}
__host__ __device__ inline int num_blocks(int Mt, int Nt, int sup_m, int sup_n) {
  int s = ((Mt + sup_m - 1) / sup_m) * ((Nt + sup_n - 1) / sup_n);
  return (s + NXCD - 1) / NXCD * NXCD * (sup_m * sup_n);
}
__device__ inline bool tile_coords(int bid, int Mt, int Nt, int sup_m, int sup_n, int& tm, int& tn, int& sm, int& sn) {
  const int sNt = (Nt + sup_n - 1) / sup_n, sMt = (Mt + sup_m - 1) / sup_m;
  const int xcd = bid % NXCD, local = bid / NXCD;
  const int q = local / (sup_m * sup_n), within = local % (sup_m * sup_n);
  const int s = q * NXCD + xcd;
  if (s >= sMt * sNt) return false;
  sm = within % sup_m; sn = within / sup_m;
  tm = (s / sNt) * sup_m + sm;
  tn = (s % sNt) * sup_n + sn;
  return tm < Mt && tn < Nt;
}

// swizzle of the K-major A panel: rows k, k+1, k+2, k+3 and k+8 (or k+16) get distinct values
__device__ inline int kswz(int k) { return (k & 3) | ((((k >> 3) ^ (k >> 4)) & 1) << 2); }

__device__ inline int min_int(int a, int b) { return a < b ? a : b; }
__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// The MFMA is issued through inline assembly with the accumulator tied in place in an
// accumulation register: left to the register allocator, a few of the 64 accumulator tuples
// (which fill the accumulation file completely) end up rotating through copies every iteration.
// The K loop issues the two 32-wide K steps of an accumulator back to back: the second MFMA reads
// as SrcC the register tuple the first one writes as vDst.  That dependent pair with identical
// SrcC / vDst is the case the hardware interlocks by itself (no software wait states required);
// no other instruction touches an accumulator inside the loop.  The first ordinary reads after
// the K loop are fenced by drain_mfma() below.
__device__ __forceinline__ void mfma16(f32x4& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// The last MFMA of a loop body whose accumulators the compiler may move behind the loop (it does, where
// paths meet): the wait states before an ordinary read of the result are part of it.
__device__ __forceinline__ void mfma16_then_wait(f32x4& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\ts_nop 15\n\ts_nop 3" : "+a"(c) : "v"(a), "v"(b));
}
// Wait states between the last MFMAs of the K loop and the first ordinary read of their
// results (the hazard checker of the compiler does not look into inline assembly).
__device__ __forceinline__ void drain_mfma(f32x4 (&r)[8]) {
  asm volatile("s_nop 15\n\ts_nop 15"
               : "+a"(r[0]), "+a"(r[1]), "+a"(r[2]), "+a"(r[3]), "+a"(r[4]), "+a"(r[5]), "+a"(r[6]), "+a"(r[7]));
}

// Lane number as the code after the K loops takes it: recomputed there from the execution mask, so
// that nothing lane-dependent has to stay alive (that is, be spilled to scratch memory) across the
// loop, whose body owns every vector register.  A reload from scratch is a vector-memory load: the wait
// for it would also wait for every store issued before it, and between the stores of the forward
// epilogue that costs microseconds each time.
__device__ __forceinline__ int lane_now() {
  int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  asm volatile("" : "+v"(l));   // opaque: what is derived from it is computed where it is used, not hoisted
  return l;
}

// Forward epilogue of a wave's 128 x (16 NJ) sub-tile: vocabulary ids from m0 + 128 wm, token columns from
// n0 + 16 NJ wn, partial sums with index pidx; target_logit(j): that of the lane's token in column block j; accumulator element (i, j, e) of a lane is vocabulary
// id vrow(i, e), token column ncol_base + 16 j.
template <int NJ, class Zt>
__device__ __forceinline__ void forward_epilogue(const Params& p, f32x4 (&acc)[8][NJ], Zt target_logit, int m0,
                                                 int n0, int pidx, int wm, int wn, int N) {
  const int lane = lane_now(), frow = lane & 15, fq = lane >> 4;
  const int ncol_base = n0 + wn * (16 * NJ) + frow;
      // rows = vocabulary ids, cols = token rows of the chunk.  Exponentials are taken relative to
      // the row's offset c2 = z_target * log2(e) + margin (log2 domain), one offset for all
      // vocabulary tiles of a row: e = 2^(z log2(e) - c2), clamped so that neither e nor any sum of
      // it can overflow.  The sums over the wave's 128 vocabulary ids are this tile's partials; e
      // itself, as bf16, is the backward pass's operand (dz = (-g / S)(e - S onehot)).
      constexpr float LOG2E = 1.4426950408889634f;
      const bool full = (m0 + wm * 128 + 128 <= p.V);
          // vocabulary id of accumulator (i, e) of this lane
      auto vrow = [&](int i, int e) {
        return m0 + wm * 128 + 32 * (i >> 1) + 8 * fq + 4 * (i & 1) + e;
      };
      // The body is instantiated for full / ragged vocabulary tiles and with / without the entropy
      // sums: both conditions are uniform, and left as run-time selects they cost four more
      // instructions per logit (row id, compare, two selects) than the six the work needs
      // (accumulator read, multiply-add, clamp, exponential, add, half a packed conversion).
      auto body = [&](auto full_tile, auto with_ez) {
        constexpr bool kFull = decltype(full_tile)::value, kEz = decltype(with_ez)::value;
  #pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int n = ncol_base + j * 16;
          const bool live = n < N;
          const float zt = target_logit(j);
          const float c2 = live ? fmaf(zt, LOG2E, kStashMargin2) : 0.f;
          uint16_t* erow = p.estash + (int64_t)n * p.lde + m0 + wm * 128 + 8 * fq;
          float s = 0.f, t = 0.f;
  #pragma unroll
          for (int q = 0; q < 4; ++q) {
            // accumulators 2q and 2q+1 hold 8 consecutive vocabulary ids of this lane
            bf16x8 h;
  #pragma unroll
            for (int u = 0; u < 2; ++u)
  #pragma unroll
              for (int e = 0; e < 4; ++e) {
                // (read where it is used: left to the compiler, the copies out of the accumulation
                // registers are hoisted to the top of the epilogue and fill the register file)
                float z;
                asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(z) : "a"(acc[2 * q + u][j][e]));
                float w = exp2_fast(fminf(fmaf(z, LOG2E, -c2), kStashClamp2));
                if (!kFull) w = vrow(2 * q + u, e) < p.V ? w : 0.f;
                s += w;
                if (kEz) t = fmaf(w, z, t);     // for the entropy: sum e * z  (H = lse - E_p[z])
                h[4 * u + e] = (__bf16)w;
              }
            if (p.estash != nullptr && live) {
              // 16 bytes per lane, the four lanes of a token row side by side (64 bytes).  Streaming
              // store (non-temporal, device scope): the stash is 5 GB per launch and is next read by
              // the backward launches, so it should not displace operand panels from the L2 and the
              // memory-side cache (2 % of the launch against a plain store).  Written in assembly
              // for its cache policy bits; the two wait states after it are the ones the hardware
              // needs before the data registers of a store wider than 8 bytes may be overwritten
              // (the compiler inserts them for its own stores only).
              asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" :: "v"(erow + 32 * q), "v"(h) : "memory");
            }
          }
          s += __shfl_xor(s, 16);
          s += __shfl_xor(s, 32);
          if (fq == 0 && live) p.part_sum[(int64_t)pidx * p.part_stride + n] = s;
          if (kEz) {
            t += __shfl_xor(t, 16);
            t += __shfl_xor(t, 32);
            if (fq == 0 && live) p.part_ez[(int64_t)pidx * p.part_stride + n] = t;
          }
          // one column block at a time: interleaving them runs the register allocator out of
          // registers, and its reloads from scratch wait for the stores issued so far
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      if (full) {
        if (p.part_ez != nullptr) body(Flag<true>{}, Flag<true>{}); else body(Flag<true>{}, Flag<false>{});
      } else {
        if (p.part_ez != nullptr) body(Flag<false>{}, Flag<true>{}); else body(Flag<false>{}, Flag<false>{});
      }
}

// ---------------------------------------------------------------------------------------------
// Forward, last column of tiles with at most 128 tokens: 256 x 128 tiles, waves 2 x 2, each 128 x 64.  A panel takes half
// the MFMAs, so the fragments of two panels fit into registers and three panels into LDS: a panel's MFMAs run
// on fragments read during the panel before, while the loads of the third next one go into the slot those left.
// The load path bounds it (48 KB per 1024 MFMA cycles): a tile takes 0.55 - 0.6 of a 256 x 256 one.  Forward launch, rows
// padded to 256 and now, us: V = 151936, d = 4096, 300 rows 565 and 506, 384 rows 554 and 481, 600 rows 739 and
// 630, 1877 rows 1859 and 1676; d = 1536, 300 rows 243 and 207, 1877 rows 798 and 764; V = 50257, d = 712, 1877 rows 184 and 175.
// The same for the dH launch's last row of tiles was slower (327 rows, d = 4096 460 -> 576 us): its panels of W come from
// memory, and the shorter panel leaves them half the time to arrive.
// The kernel's arguments are read again behind the branch: kept alive across both paths they cost scalar
// spills that slowed every tile (d = 712: 3 %).
// ---------------------------------------------------------------------------------------------
constexpr int HALF_COLS = 128;
constexpr int HALF_STAGE = TILE_BYTES + TILE_BYTES / 2, HALF_PIPE = 3 * HALF_STAGE;   // A and half as much B, 48 KB
constexpr int HALF_LOADS = 12;                                      // direct loads per wave and panel: 8 of A, 4 of B

__device__ __forceinline__ void half_column_tile(unsigned char* smem, int tm, int n0, int N) {
  typedef const __attribute__((address_space(4))) Params* KernArg;
  KernArg arg = (KernArg)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(arg));
  const Params& p = *(const Params*)arg;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1, frow = lane & 15, fq = lane >> 4;
  const int m0 = tm * BM, M = p.M, nk = p.K / BK;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  // panels, swizzles and fragment rows as in the full tile
  const uint16_t* src[HALF_LOADS];
#pragma unroll
  for (int i = 0; i < HALF_LOADS; ++i) {
    const bool a = i < 8;
    const int r = (a ? wave * 8 + i : wave * 4 + i - 8) * 8 + (lane >> 3);
    const int row = a ? (m0 + r < M ? m0 + r : M - 1) : (n0 + r < N ? n0 + r : N - 1);
    const int swz = a ? ((r >> 1) & 1) | (((r >> 3) & 3) << 1) : (r >> 1) & 7;
    src[i] = (a ? p.A + (int64_t)row * p.lda : p.B + (int64_t)row * p.ldb) + ((lane & 7) ^ swz) * 8;
  }
  const uint32_t lds_a = __builtin_amdgcn_readfirstlane(lds_base + wave * 8192);
  const uint32_t lds_b = __builtin_amdgcn_readfirstlane(lds_base + TILE_BYTES + wave * 4096);
  // load l of panel kt (behind the end: the last one again, into a slot nobody reads)
  auto load = [&](int l, int kt, uint32_t stage) {
    kt = kt < nk ? kt : nk - 1;
    const int64_t off = (int64_t)kt * (BK * 2) + (l < 8 && kt >= p.a_tail_panel ? p.a_tail_delta : 0);
    const uint32_t lds = (l < 8 ? lds_a + l * 1024 : lds_b + (l - 8) * 1024) + stage;
    uint64_t addr;
    asm volatile("s_mov_b32 m0, %3\n\tv_lshl_add_u64 %0, %1, 0, %2\n\tglobal_load_lds_dwordx4 %0, off"
                 : "=&v"(addr) : "v"(src[l]), "s"(off), "s"(lds) : "memory");
  };
  int a_off[2], b_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int chunk = (ks << 2) | fq;
    a_off[ks] = (wm * 128 + 8 * (frow >> 2) + (frow & 3)) * 128 + ((chunk ^ (((frow >> 1) & 1) | ((frow >> 2) << 1))) << 4);
    b_off[ks] = TILE_BYTES + (wn * 64 + frow) * 128 + ((chunk ^ ((frow >> 1) & 7)) << 4);
  }
  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  bf16x8 fa[2][8][2], fb[2][4][2];                    // [this panel / the next][block][K step]
  // fragment n of a panel: the 8 of B first
  auto read = [&](int set, uint32_t stage, int n) {
    if (n < 8) fb[set][n / 2][n & 1] = *reinterpret_cast<const bf16x8*>(smem + stage + b_off[n & 1] + (n / 2) * 2048);
    else fa[set][(n - 8) / 2][n & 1] = *reinterpret_cast<const bf16x8*>(smem + stage + a_off[n & 1] + ((n - 8) >> 2) * 4096 + (((n - 8) >> 1) & 1) * 512);
  };
  // 64 MFMAs, between them one piece at a time: a load, two fragments, a load, ...  The barrier: every wave has the
  // fragments of this panel in registers (its slot can be refilled), and the next panel has landed (only the
  // loads of the one behind it are outstanding).
  auto panel = [&](auto second, int kt, uint32_t st_this, uint32_t st_next) {
    constexpr int set = decltype(second)::value ? 1 : 0;
    constexpr int kPieces = 3 * HALF_LOADS, kFirst = 3, kSlots = 54;
#pragma unroll
    for (int m = 0; m < 64; ++m) {
      const int g = m / 8, j = m / 2 % 4, ks = m & 1;
      if (set == 1 && m == 63) mfma16_then_wait(acc[g][j], fa[set][g][ks], fb[set][j][ks]);
      else mfma16(acc[g][j], fa[set][g][ks], fb[set][j][ks]);
      if (m == kFirst - 1) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(HALF_LOADS) & ~(15 << 8));   // (and no LDS read)
        __syncthreads();
      }
      if (m >= kFirst && m < kFirst + kSlots) {
        const int n = m - kFirst, q = n * kPieces / kSlots;
        if (n == 0 || q != (n - 1) * kPieces / kSlots) {
          if (q % 3 == 0) load(q / 3, kt + 3, st_this); else read(set ^ 1, st_next, q - q / 3 - 1);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  {
    int n = n0 + wave * 64 + lane; n = n < N ? n : N - 1;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :: "v"(p.zt + n), "s"(__builtin_amdgcn_readfirstlane(lds_base + HALF_PIPE + wave * 256)) : "memory");
  }
#pragma unroll
  for (int s = 0; s < 3; ++s)
#pragma unroll
    for (int l = 0; l < HALF_LOADS; ++l) load(l, s, s * HALF_STAGE);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * HALF_LOADS));
  __syncthreads();
#pragma unroll
  for (int n = 0; n < 24; ++n) read(0, 0, n);
  uint32_t st = 0;
  auto next = [](uint32_t x) { return x == 2 * HALF_STAGE ? 0u : x + HALF_STAGE; };
  int kt = 0;
  do {                                                // (an even number of panels, at least two)
    panel(Flag<false>{}, kt, st, next(st));
    st = next(st);
    panel(Flag<true>{}, kt + 1, st, next(st));
    st = next(st);
    kt += 2;
  } while (kt < nk);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));          // no direct load may outlive the wave
  const unsigned char* const zt_lds = smem + HALF_PIPE + ((wn * 64 + (lane_now() & 15)) << 2);
  forward_epilogue<4>(p, acc, [&](int j) { return *reinterpret_cast<const float*>(zt_lds + j * 64); }, m0, n0, tm * 2 + wm, wm, wn, N);
}

template <int MODE>
__global__ __launch_bounds__(NTHREADS) void gemm_nt_bf16(Params p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);

  // valid rows of this chunk (device-side, no host sync)
  int64_t nv64 = *p.n_scored - p.chunk_start;
  const int nvalid = nv64 < 0 ? 0 : (nv64 > p.chunk_rows ? p.chunk_rows : (int)nv64);

  int M = p.M, N = p.N, K = p.K;
  if (MODE == MODE_FWD) N = nvalid;
  if (MODE == MODE_DH) M = nvalid;
  if (MODE == MODE_DW) K = dw_panels(nvalid, K) * BK;
  if (MODE == MODE_FWD && nvalid == 0) return;
  if (MODE == MODE_DH && nvalid == 0) return;
  if (MODE == MODE_DW && nvalid == 0 && !p.overwrite) return;

  const int Mt = (M + BM - 1) / BM, Nt = (N + BN - 1) / BN;
  int tm, tn;
  int sm, sn, sup_m, sup_n;        // position of the tile among those that share its panels
  int k_first = 0;                 // first K panel of this workgroup (tail slices start later)
  float* tail_out = nullptr;       // DH / DW tail slice: where the accumulators go instead
  if (MODE != MODE_DW) {
    int bid = blockIdx.x, split = 1, slice = 0;
    const int tiles = Mt * Nt, whole = tiles / kRound * kRound;
    if (MODE == MODE_DH && bid >= whole) {
      const int rest = tiles - whole;
      split = dh_split(rest, K / BK, p.max_items);
      if (split > 1) {
        // an XCD takes consecutive items, i.e. mostly tiles of one slice
        const int items = rest * split, per = (items + NXCD - 1) / NXCD;
        const int e = bid - whole, item = e % NXCD * per + e / NXCD;
        if (e / NXCD >= per || item >= items) return;
        slice = item / rest;
        tile_at(whole + item - slice * rest, Mt, Nt, tm, tn);
        const int nk_all = K / BK, per_slice = slice_panels(nk_all, split);
        k_first = slice * per_slice;
        const int k_end = k_first + per_slice < nk_all ? k_first + per_slice : nk_all;
        K = k_end > k_first ? (k_end - k_first) * BK : 0;
        tail_out = p.tail_part + (int64_t)item * (BM * BN);
      }
    }
    if (split == 1 && !dealt_tile(bid, Mt, Nt, tm, tn)) return;
    sm = tm % kBand; sn = tn % 4; sup_m = kBand; sup_n = 4;
  } else if (p.tail_split > 0) {
    sup_m = p.sup_m; sup_n = p.sup_n;
    if ((int)blockIdx.x < p.main_blocks) {
      if (!tile_coords(blockIdx.x, p.tail_m0, Nt, p.sup_m, p.sup_n, tm, tn, sm, sn)) return;
    } else {
      // one XCD takes consecutive items (the host says how many: the XCDs that the whole tiles
      // leave idle earlier take more), i.e. mostly tiles of one slice: they walk the same K range
      // and share its operand panels in that L2
      const int e = blockIdx.x - p.main_blocks;
      const int tiles = p.tail_rows * Nt;
      const int item = p.tail_first[e % NXCD] + e / NXCD;
      if (item >= p.tail_first[e % NXCD + 1]) return;
      const int slice = item / tiles, t = item % tiles;
      sm = t / Nt; sn = t % Nt;
      tm = p.tail_m0 + sm; tn = sn;
      const int nk_all = K / BK, per = slice_panels(nk_all, p.tail_split);
      k_first = slice * per;
      if (slice >= slices_in_use(nk_all, p.tail_split)) return;   // empty: nothing to store, and nobody reads it
      const int k_end = k_first + per < nk_all ? k_first + per : nk_all;
      K = k_end > k_first ? (k_end - k_first) * BK : 0;
      tail_out = p.tail_part + (int64_t)item * (BM * BN);
    }
  } else {
    sup_m = p.sup_m; sup_n = p.sup_n;
    if (!tile_coords(blockIdx.x, Mt, Nt, sup_m, sup_n, tm, tn, sm, sn)) return;
  }
  if (MODE == MODE_FWD && __builtin_expect(N - (Nt - 1) * BN <= HALF_COLS, 0)) {
    // A last column of at most 128 tokens takes half tiles.  They are dealt like the others, to every XCD its share: the
    // columns of a band start at another one in every band (with 8 columns, XCDs would else have all of them or none).
    int columns = Nt;
    asm volatile("" : "+s"(columns));                 // (the division stays in this branch)
    tn += tm / kBand % columns;
    tn = tn < Nt ? tn : tn - Nt;
    if (tn == Nt - 1) { half_column_tile(smem, tm, tn * BN, N); return; }
  }
  const int m0 = tm * BM, n0 = tn * BN;

  // ---- global -> LDS: one direct load moves 1 KB, contiguous in LDS.
  // Row-major operands ([row][k], k contiguous): 8 rows x 128 B per load.  Wave w owns row
  // blocks 8w .. 8w+7 of each operand panel; lane l fills LDS chunk (row l/8, slot l%8) and
  // therefore fetches logical chunk slot ^ ((row >> 1) & 7).
  // K-major operands (DW: A[m][k] = dz[k][m], stored as token rows with the vocabulary contiguous;
  // DH: B[n][k] = W[k][n], the rows of W): the panel is 64 k rows x 512 B and a load moves 2 of them; lane l fills chunk
  // slot l%32 of row l/32 and fetches logical chunk slot ^ (h(k) << 1), the swizzle that makes
  // the transposing fragment reads below conflict-free.
  constexpr bool A_KMAJOR = (MODE == MODE_DW);
  constexpr bool B_KMAJOR = (MODE == MODE_DH);
  // FWD: the 16 rows of A fragment i are not 16 consecutive panel rows but
  //   rho(i, r) = 32*(i/2) + 8*(r/4) + 4*(i%2) + r%4      (within the wave's 128 rows),
  // so that a lane's accumulators (i = 2t, 2t+1; e = 0..3) are 8 consecutive vocabulary ids
  // and the bf16 stash of exponentials can be stored from registers, 16 bytes per lane, without an LDS round
  // trip.  The chunk swizzle of the A panel then takes row bits 1, 3, 4 (the ones that vary
  // inside a fragment) instead of bits 1-3.
  constexpr bool A_PERM = (MODE == MODE_FWD);
  const int64_t a_kstep = A_KMAJOR ? (int64_t)BK * p.lda : BK;   // elements per K panel
  const int lrow = lane >> 3;
  const uint16_t* a_ptr[8];
  const uint16_t* b_ptr[8];
  uint32_t b_voff[8];                                 // DH: byte offset of the lane's chunk from the wave's 16 rows of W
  // Workgroups that share a panel (same sm for A, same sn for B) walk its row blocks in a
  // different cyclic order (rot_a, rot_b), so that they do not all ask the L2 for the same lines
  // at the same moment (1-2 % on the forward and dH launches).
  uint32_t lds_a[8], lds_b[8];                        // LDS offset of load i within the wave's 8 KB
  const float* zt_ptr = nullptr;                      // forward: this lane's entry of the tile's target logits
  {
    const int rot_a = (sn * 8 / sup_n) & 7, rot_b = (sm * 8 / sup_m) & 7;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int ia = (i + rot_a) & 7, ib = (i + rot_b) & 7;
      lds_a[i] = __builtin_amdgcn_readfirstlane(ia * 1024);
      lds_b[i] = __builtin_amdgcn_readfirstlane(ib * 1024);
      const int r = (wave * 8 + ia) * 8 + lrow;         // row within the 256-row panel
      const int rB = (wave * 8 + ib) * 8 + lrow;
      const int lchunk = (lane & 7) ^ ((rB >> 1) & 7);
      const int lchunk_a = A_PERM ? ((lane & 7) ^ (((r >> 1) & 1) | (((r >> 3) & 3) << 1))) : ((lane & 7) ^ ((r >> 1) & 7));
      int ra = m0 + r; ra = ra < M ? ra : M - 1;
      int rb = n0 + rB; rb = rb < N ? rb : N - 1;
      int64_t rowa = ra, rowb = rb;
      if (A_KMAJOR) {
        const int k = 2 * (wave * 8 + ia) + (lane >> 5);  // k row within the panel
        // (columns from V on, whose products are not stored, come from the tile's first chunk again: the pad
        // columns of the stash are written past the caches and no other launch reads them, and with few tiles
        // this one lasts as long as the tile that fetches them: 41444 rows, V = 329, d = 240 924 us, now 671)
        const int col = m0 + (((lane & 31) ^ (kswz(k) << 1)) << 3);
        a_ptr[i] = p.A + ((int64_t)k_first * BK + k) * p.lda + (col < p.V ? col : m0);
      } else {
        a_ptr[i] = p.A + rowa * p.lda + lchunk_a * 8 + (MODE == MODE_DH ? k_first * BK : 0);
      }
      if (B_KMAJOR) {
        const int k = 2 * ib + (lane >> 5);
        b_voff[i] = (uint32_t)k * (uint32_t)(p.ldb * 2) + (((lane & 31) ^ (kswz(wave * 16 + k) << 1)) << 4);
      } else b_ptr[i] = p.B + rowb * p.ldb + lchunk * 8 + (MODE == MODE_DW ? k_first * BK : 0);
    }
    if (MODE == MODE_FWD) {
      int n = n0 + wave * 64 + lane; n = n < N ? n : N - 1;
      zt_ptr = p.zt + n;
    }
  }
  // The direct load is issued through inline assembly on purpose: the compiler's wait-count
  // pass treats a global load that writes LDS as touching both address spaces and then
  // drains every counter to zero before each LDS read, which serialises the pipeline.
  // Issued this way the loads are invisible to that pass; their completion is awaited
  // explicitly below with s_waitcnt vmcnt(0) before the barrier that publishes a panel.
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(lds_base + wave * 8192);

  // forward: the tile's 256 target logits travel to LDS with the tile's first panel (4 bytes per
  // lane, one direct load per wave) and are published by the same barrier, so that the epilogue
  // starts without a round trip to global memory
  auto issue_zt = [&]() {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :: "v"(zt_ptr), "s"(__builtin_amdgcn_readfirstlane(lds_base + PIPE_BYTES + wave * 256))
                 : "memory");
  };

  // ---- fragment read offsets.  A 16x16x32 operand fragment: lane -> row (lane & 15),
  // 16-byte K chunk (lane >> 4) of a 32-wide K step.  A 128-bit LDS read is served 16 lanes
  // per cycle over 64 banks; rows 2 apart share a bank window (128-byte rows), the swizzle
  // (row / 2) % 8 spreads the 16 rows of a fragment over distinct banks.
  const int frow = lane & 15, fq = lane >> 4;
  int a_off[2], b_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int chunk = ((ks << 2) | fq) ^ ((frow >> 1) & 7);
    if (A_PERM) {
      const int chunk_a = ((ks << 2) | fq) ^ (((frow >> 1) & 1) | ((frow >> 2) << 1));
      a_off[ks] = (wm * 128 + 8 * (frow >> 2) + (frow & 3)) * 128 + (chunk_a << 4);
    } else {
      a_off[ks] = (wm * 128 + frow) * 128 + (chunk << 4);
    }
    b_off[ks] = TILE_BYTES + (wn * 128 + frow) * 128 + (chunk << 4);
  }

  // K-major panel: the transposing LDS read hands lane (g = lane / 16, s = lane % 16) the four
  // k values kb .. kb+3 of column m = mb + s when lane s points at row kb + s/4, columns
  // mb + 4*(s%4) .. +3.  Two of them (kb = 8g and 8g + 4 within the K step) make the lane's
  // 8-element fragment.  A 64-bit read is served 32 lanes per cycle: 8 rows x 32 bytes, and the
  // swizzle h(k) moves the 32-byte column groups of those rows to distinct bank windows.
  int a_tr_base = 0, b_tr_base = 0;
  {
    const int k = 8 * fq + (frow >> 2);
    const int base = k * 512 + (kswz(k) << 5) + ((frow & 2) << 3) + ((frow & 1) << 3);
    if (A_KMAJOR) a_tr_base = base + wm * 256;
    if (B_KMAJOR) b_tr_base = base + wn * 256;
  }
  auto read_kmajor = [&](int off) -> bf16x8 {
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4i16* lds_v4i16;
    unsigned char* q = smem + off;
    const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)q);
    const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(q + 2048));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto read_a = [&](int st, int ks, int ib) -> bf16x8 {
    if (A_KMAJOR) return read_kmajor(st + (a_tr_base ^ (ib << 5)) + ks * 16384);
    return *reinterpret_cast<const bf16x8*>(smem + st + a_off[ks] +
                                            (A_PERM ? (ib >> 1) * 4096 + (ib & 1) * 512 : ib * 2048));
  };

  f32x4 acc[8][8];
  const int nk = K / BK;
  // Software pipeline.  Panel kt+1 is loaded during the MFMAs of panel kt (double buffer).
  // A panel is 8 groups; group g multiplies the A fragments of 16-row block g (both 32-wide
  // K steps) with the panel's 16 B fragments: 16 MFMAs, the two K steps of an accumulator back
  // to back.  Keeping an accumulator for two consecutive MFMAs costs measurably less energy than
  // touching 64 different ones in turn (about 5 % more FLOP/s from an MFMA-only loop at the
  // power limit), which is what bounds these kernels on real data.
  // Registers: the B fragments of a whole panel stay resident, in two sets (this panel / the
  // next one); A fragments sit in a ring of four pairs.  The schedule of reads, barrier and
  // direct loads around the MFMAs is described at `side` below.
  // The loop body (two panels, so that the B sets have fixed registers) is branch-free; loads
  // that would run past the end re-fetch the last panel into a slot nobody reads.
  bf16x8 fbx[2][2][8];   // [set][K step][16-column block]
  bf16x8 fax[4][2];      // [ring slot][K step]
  auto read_b = [&](int st, int ks, int j) -> bf16x8 {
    if (B_KMAJOR) return read_kmajor(st + TILE_BYTES + (b_tr_base ^ (j << 5)) + ks * 16384);
    return *reinterpret_cast<const bf16x8*>(smem + st + b_off[ks] + j * 2048);
  };
  // One load of the K loop: three instructions, what one MFMA leaves room for.  The address
  // arithmetic (panel offset, uniform) is part of the piece, and it separates the write of M0
  // from the load that reads it (one wait state).
  auto load_lds16_at = [](const uint16_t* base, int64_t byte_off, uint32_t lds_addr) {
    uint64_t addr;
    asm volatile("s_mov_b32 m0, %3\n\tv_lshl_add_u64 %0, %1, 0, %2\n\tglobal_load_lds_dwordx4 %0, off"
                 : "=&v"(addr) : "v"(base), "s"(byte_off), "s"(lds_addr) : "memory");
  };
  // DH: the wave's 16 rows of W in the panel being loaded, as a buffer descriptor that ends with row
  // V - 1: the contraction runs over the vocabulary rounded up to whole panel pairs, and loads
  // beyond the descriptor's end return zeros (the stash columns there are zeros as well).  w_advance
  // moves it on by a panel.
  uint64_t w_addr = 0;
  int w_left = 0;                                     // rows of W from the wave's first one on
  u32x4 w_desc = {0, 0, 0, 0x00020000u};
  auto w_set = [&]() {
    const int rows = min_int(w_left, 16);             // (below 2^25 bytes: ldb is at most 2^20)
    const int bytes = rows * (int)(p.ldb * 2) - n0 * 2;
    w_desc[0] = (uint32_t)w_addr; w_desc[1] = (uint32_t)(w_addr >> 32);
    w_desc[2] = (uint32_t)(bytes > 0 ? bytes : 0);
  };
  auto w_advance = [&]() { w_addr += (uint64_t)p.ldb * (BK * 2); w_left -= BK; w_set(); };
  if (B_KMAJOR) {
    const int64_t first = (int64_t)k_first * BK + wave_u * 16;
    w_addr = (uint64_t)(p.B + first * p.ldb + n0);
    w_left = p.V - (int)first;
    w_set();
  }
  auto load_lds16_w = [](uint32_t voff, const u32x4& desc, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
                 :: "v"(voff), "s"(desc), "s"(lds_addr) : "memory");
  };
  auto issue_range = [&](int kt, int slot, int j0, int j1) {
    const int64_t a_off = (int64_t)kt * a_kstep * 2 + (MODE == MODE_FWD && kt >= p.a_tail_panel ? p.a_tail_delta : 0);
#pragma unroll
    for (int j = j0; j < j1; ++j) {
      const uint32_t st = slot * STAGE_BYTES + wave_lds;
      if (B_KMAJOR && (j & 1)) load_lds16_w(b_voff[j >> 1], w_desc, st + TILE_BYTES + lds_b[j >> 1]);
      else if (j & 1) load_lds16_at(b_ptr[j >> 1], (int64_t)kt * (BK * 2), st + TILE_BYTES + lds_b[j >> 1]);
      else load_lds16_at(a_ptr[j >> 1], a_off, st + lds_a[j >> 1]);
    }
  };
  // One panel = 8 groups of 16 MFMAs.  A wave issues in order and the matrix pipe takes a new MFMA
  // only every 16 cycles, so whatever stands between two MFMAs in the instruction stream is free
  // as long as it fits the 12 issue cycles the pipe leaves over - and costs pipe time when it
  // comes as a block after the sixteenth.  The side work of a panel (fragment reads, the barrier,
  // direct loads with their address arithmetic) is therefore cut into pieces of one to four
  // instructions, one piece after an MFMA, in source order (both are volatile assembly or fenced):
  //   group 0      : A fragments of row block 3 (this panel); the last loads of the NEXT panel's slot
  //   groups 1 - 4 : A fragments of row blocks 4 - 7
  //   group 5      : wait for this thread's part of panel kt+1, barrier (every wave has issued its
  //                  last read of this panel's slot by then, so the slot can be refilled; panel
  //                  kt+1 becomes visible); next panel's A block 0, B column blocks 0 - 2; the first
  //                  loads of panel kt+2 into this panel's slot
  //   group 6      : next A block 1, B blocks 3 - 5, loads
  //   group 7      : next A block 2, B blocks 6 - 7, loads   (the rest follows in group 0 of the
  //                  next panel; kLoadsInGroup says how many where)
  // A fragments sit in a ring of four pairs: group g multiplies ring slot g % 4, and the slot a
  // group has just finished with is refilled during the next group.  Four loads per group over
  // four groups measured best: packing them into groups 5 - 7 costs 2 - 4 % (the load path of a
  // compute unit takes about 23 cycles per 1 KB load, four waves issuing one every 16 cycles run
  // its queue full and stall their MFMAs with it), spreading them further leaves the late ones
  // too little time to land.
  auto side = [&](int g, int m, int set, int st_cur, int st_nxt, int kt_nxt, int slot_nxt, int kt_load, int slot_cur) {
    // pieces before the loads: the barrier (group 5) and the fragment reads
    int nr = 2;
    if (g == 0) {
      if (m < 2) fax[3][m] = read_a(st_cur, m, 3);
    } else if (g <= 4) {
      if (m < 2) fax[(g - 1) & 3][m] = read_a(st_cur, m, g + 3);
      if (B_KMAJOR && g == 4 && m == 6) w_advance();
    } else {
      const int q = g - 5;                          // 0, 1, 2
      if (g == 5 && m == 0) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        __syncthreads();
      }
      if (m >= 1 && m < 3) fax[q][m - 1] = read_a(st_nxt, m - 1, q);
      const int nb = q == 2 ? 2 : 3;                // B column blocks read in this group
      if (m >= 3 && m < 3 + 2 * nb) { const int j = 3 * q + (m - 3) / 2, ks = (m - 3) & 1; fbx[set ^ 1][ks][j] = read_b(st_nxt, ks, j); }
      nr = 3 + 2 * nb;
    }
    // this group's share of the 16 loads that fill a slot, spread over the remaining gaps
    const int nl = kLoadsInGroup[g];
    if (nl > 0 && m >= nr) {
      const int room = 16 - nr;
#pragma unroll
      for (int i = 0; i < nl; ++i)
        if (m == nr + i * room / nl) {
          const int l = load_index_base(g) + i;
          if (g >= 5) issue_range(kt_load, slot_cur, l, l + 1);
          else issue_range(kt_nxt, slot_nxt, l, l + 1);
        }
    }
  };
  auto panel = [&](int set, int st_cur, int st_nxt, int kt_nxt, int slot_nxt, int kt_load, int slot_cur) {
#pragma unroll
    for (int g = 0; g < 8; ++g) {
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        // (DW: operands swapped, the accumulator holds the transposed 16 x 16 block)
        if (MODE == MODE_DW) mfma16(acc[g][m >> 1], fbx[set][m & 1][m >> 1], fax[g & 3][m & 1]);
        else mfma16(acc[g][m >> 1], fax[g & 3][m & 1], fbx[set][m & 1][m >> 1]);
        side(g, m, set, st_cur, st_nxt, kt_nxt, slot_nxt, kt_load, slot_cur);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  auto last_k = [&](int k) { return k < nk ? k : nk - 1; };
  // The number of panels is even (the launchers see to it), so that the two-panel body is the
  // only code that touches the accumulators: there is no peeled tail whose different register
  // assignment would make the compiler move accumulators around next to MFMAs it cannot see
  // into.  The last two panels read ahead and load like any other (the panel after the last is
  // a re-fetch of the last one, read into registers nobody uses).
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  if (nk > 0) {
    issue_range(0, 0, 0, 16);
    if (B_KMAJOR) w_advance();
    if (MODE == MODE_FWD) issue_zt();
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __syncthreads();
    issue_range(last_k(1), 1, 0, 16 - kLoadsCarriedOver);   // the rest comes with the first groups of the first panel
#pragma unroll
    for (int j = 0; j < 8; ++j) { fbx[0][0][j] = read_b(0, 0, j); fbx[0][1][j] = read_b(0, 1, j); }
#pragma unroll
    for (int i = 0; i < 3; ++i) { fax[i][0] = read_a(0, 0, i); fax[i][1] = read_a(0, 1, i); }
    for (int kt = 0; kt < nk; kt += 2) {
      panel(0, 0, STAGE_BYTES, last_k(kt + 1), 1, last_k(kt + 2), 0);
      panel(1, STAGE_BYTES, 0, last_k(kt + 2), 0, last_k(kt + 3), 1);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));   // no direct load may outlive the wave
    drain_mfma(acc[7]);
  }

  // ---- epilogues.  Accumulator element (i, j, e) of this lane is
  //   row m = m0 + wm*128 + i*16 + 4*(lane>>4) + e      (FWD: the permuted row, see vrow below)
  //   col n = n0 + wn*128 + j*16 + (lane & 15)
  // (DW: row m = m0 + wm*128 + i*16 + (lane & 15), col n = n0 + wn*128 + j*16 + 4*(lane>>4) + e)
  if (MODE == MODE_DH) __syncthreads();   // its staged epilogue reuses the panels' LDS

  if (MODE == MODE_FWD) {
    const unsigned char* const zt_lds = smem + PIPE_BYTES + (((wave_u & 1) * 128 + (lane_now() & 15)) << 2);
    forward_epilogue<8>(p, acc, [&](int j) { return *reinterpret_cast<const float*>(zt_lds + j * 64); }, m0, n0,
                        tm * 2 + (wave_u >> 1), wave_u >> 1, wave_u & 1, N);
  } else if (MODE == MODE_DH) {
    const int lane = lane_now(), wave = wave_u, tid = wave * 64 + lane;
    const int wm = wave >> 1, wn = wave & 1, frow = lane & 15, fq = lane >> 4;
    const int mrow_base = m0 + wm * 128 + 4 * fq;
    const int ncol_base = n0 + wn * 128 + frow;
    // rows = token rows of the chunk (scattered to their slots), cols = hidden index; a row
    // of the stash times W is the row's dz W up to its scale -g / S, applied here
    // an accumulator, read where it is used on all three paths: left to the compiler, the copies out of the
    // accumulation registers are hoisted above the branches and 13 of them spilled to scratch memory behind
    // every tile's K loop (16384 rows, d = 1024, V = 512, no dW: float output 188.4 us a call, now 182.9;
    // bf16 output 165.2 and 163.6)
    auto read_acc = [&](int i, int j, int e) {
      float x;
      asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(x) : "a"(acc[i][j][e]));
      return x;
    };
    if (tail_out != nullptr) {
      // a slice of the contraction: the accumulators as they are, [256][256] fp32
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float* row = tail_out + (wm * 128 + i * 16 + 4 * fq + e) * BN + wn * 128 + frow;
#pragma unroll
          for (int j = 0; j < 8; ++j) row[j * 16] = read_acc(i, j, e);
        }
    } else if (p.dh_f32) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = mrow_base + i * 16 + e;
          if (m < M) {
            const float sc = p.row_scale[m];
            float* row = reinterpret_cast<float*>(p.dH) + (int64_t)p.row_index[m] * p.d;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int n = ncol_base + j * 16;
              const float x = read_acc(i, j, e);
              if (n < p.d) row[n] = sc * x;
            }
          }
        }
    } else {
      // stage the tile as bf16 in LDS, [token][hidden], then 32 lanes store one 512-byte row segment
      __bf16* st = reinterpret_cast<__bf16*>(smem);
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int m = mrow_base + i * 16 + e;
          const float sc = p.row_scale[m < M ? m : M - 1];
#pragma unroll
          for (int j = 0; j < 8; ++j)
            st[(wm * 128 + i * 16 + 4 * fq + e) * DHSTAGE_LD + wn * 128 + j * 16 + frow] = (__bf16)(sc * read_acc(i, j, e));
        }
      __syncthreads();
#pragma unroll 4
      for (int k = 0; k < 32; ++k) {
        const int c = tid + NTHREADS * k;
        const int row = c >> 5, col = c & 31;
        if (m0 + row < M && n0 + col * 8 < p.d) {
          const u32x4 v = *reinterpret_cast<const u32x4*>(smem + row * (DHSTAGE_LD * 2) + col * 16);
          *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(p.dH) + (int64_t)p.row_index[m0 + row] * p.d + n0 + col * 8) = v;
        }
      }
    }
  } else {
    const int lane = lane_now(), wave = wave_u;
    const int wm = wave >> 1, wn = wave & 1, frow = lane & 15, fq = lane >> 4;
    // rows = vocabulary ids, cols = hidden index; fp32 accumulate into dW.  With the operands swapped a
    // lane holds four consecutive columns of a row, so that dW is read and written 16 bytes at a
    // time (d is a multiple of 8; with 4-byte accesses the launch took 1128 instead of 1023 us for 512 rows,
    // V = 151936, d = 4096, and 127 instead of 109 for V = 32000, d = 2048).  The old values of one 16-row band
    // are fetched as a batch before any store, so their latencies overlap.
    // A K slice of a tail tile stores its partial tile as it is, [256][256] fp32, to the scratch
    // area instead (dw_tail_reduce adds the slices in their order): the same code with the
    // tile's own origin, row stride and bounds.
    const bool tail = tail_out != nullptr;
    float* const dst = tail ? tail_out : p.dW;
    const int64_t ld = tail ? BN : p.d;
    const int v_org = tail ? m0 : 0, n_org = tail ? n0 : 0;
    const int v_end = tail ? m0 + BM : p.V, n_end = tail ? n0 + BN : p.d;
    const bool overwrite = tail || p.overwrite;
    const int vbase = m0 + wm * 128 + frow, nbase = n0 + wn * 128 + 4 * fq;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int v = vbase + i * 16;
      float* const row = dst + (int64_t)((v < v_end ? v : v_end - 1) - v_org) * ld - n_org;
      f32x4 old[8];
      if (!overwrite) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int n = nbase + j * 16;
          old[j] = *reinterpret_cast<const f32x4_any*>(row + (n < n_end ? n : n_end - 4));
        }
      }
      if (v < v_end) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int n = nbase + j * 16;
          f32x4 x = acc[i][j];
          if (!overwrite) x = old[j] + x;
          if (n < n_end) *reinterpret_cast<f32x4_any*>(row + n) = x;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Forward of at most 256 rows: 128 x 256 tiles (vocabulary x tokens), two workgroups per compute unit.
// With a single tile column every panel of W is read once, and the launch is bound by how fast W
// streams in and by its last round: 594 tiles of 256 x 256 are three rounds of 256 for 2.3 rounds'
// work, and one workgroup per compute unit has one panel of W in flight and nothing to do behind its
// epilogue.  Tiles half as high let two workgroups share a compute unit (80 KB of LDS, 216 registers each).
// The L2 takes one request per clock and channel, of 64 or of 128 bytes: with both operands fetched in
// 64-byte pieces (32 K-elements of a row) the launch was bound by those requests.  W comes in chunks of 64
// K-elements, two steps of the loop, and the token rows lie in blocks of 32 columns ([dp / 32][rows][32],
// written that way by the row preparation), so that both are fetched in whole lines.  Waves without tokens
// only load their share of W.  Every tile walks K from column 0, as the large tile does: a logit's products are
// added in one order in every forward kernel, and a token's scores have the same bits in a pass of any length.
// Rows of a power of two of bytes lie on the same L2 and memory channels, and tiles that are all at one column ask the
// same channels at the same time.  Tiles that each start at another column avoid that but give other bits than the
// large tile; instead the first tile of every place on the chip starts up to 31 x 2048 clocks late, by its number among the tiles of
// its XCD, and those behind it stay apart.  Scoring call, us, at once and one after another: V = 151936, d = 4096, 1 row
// 310 and 264, 64 rows 318 and 274, 128 rows 317 and 293; d = 2048 162 and 139, 169 and 143, 181 and 163; V = 65536,
// d = 4096 145 and 126, 147 and 127, 144 and 134; V = 128256, d = 8192 434 and 418, 418 and 418, 455 and 437.  Where the
// MFMAs bind, or the launch is too short for the delay, it costs: 201 rows, V = 151936, d = 4096 341 and 344, d = 2048 186
// and 194; one round of short tiles (V = 65536, d = 2048) 51 and 69; half a round (V = 34000, d = 4096) 72 and 92; rows of
// 12 KB, 128 rows 342 and 357, of 32 KB, V = 34000, 1 row 256 and 285.  Hence the bounds: rows of 4, 8 and 16 KB, two waves with
// tokens at most, more than half of the places taken, at least 48 chunks of W per place (V = 50000, d = 4096, where that
// lies: 1 row 110 and 102, 128 rows 114 and 121).
// Scoring call, us, 256 x 256 tiles, these in 64-byte pieces, now: V = 151936, d = 4096, 64 rows 367, 315 and 274,
// 128 rows 377, 348 and 293, 201 rows 387, 395 and 334, 256 rows 408, 412 and 340; d = 1536 154, 132 and 113, 158, 143
// and 115, 164, 162 and 138, 172, 162 and 140; V = 32000, d = 2048, 256 rows 53, 52 and 45.
// The line lies at one tile column because the load path of a compute unit (23 clocks per
// KB) then has to deliver 24 KB per 512 MFMA cycles: used for every column, 4096 rows, d = 1536 / 2048 / 4096
// take 1830 / 1876 / 4163 us in the launch against 1740 / 1769 / 3805 with the large tile.  The rows that count are
// slots (rounded up to 256), the scored ones being known on the device only.
// ---------------------------------------------------------------------------------------------
constexpr int FM = 128, FN = kFewRows, FK = kRowBlock;
constexpr int F_CHUNK = FM * BK * 2, F_STAGE = FN * FK * 2;         // 16 KB: 64 K-elements of W; 16 KB: 32 of the tokens
constexpr int F_CHUNKS = 2, F_STAGES = 3;
constexpr int F_B = F_CHUNKS * F_CHUNK, F_LDS = F_B + F_STAGES * F_STAGE;
constexpr int F_LOADS = 4;                                          // direct loads per wave and chunk, or stage
constexpr int F_PLACES = 512;                                       // workgroups on the chip at a time

__global__ __launch_bounds__(NTHREADS, 2) void forward_few_bf16(Params p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int frow = lane & 15, fq = lane >> 4;
  int64_t nv64 = *p.n_scored - p.chunk_start;
  const int N = nv64 < 0 ? 0 : (nv64 > p.chunk_rows ? p.chunk_rows : (int)nv64);
  if (N == 0) return;
  // one column of tiles over whole 256-wide pairs of them, so that every partial sum and every pad
  // column of the stash is written; in order: all tiles share the token rows, and runs of 64 tiles per XCD
  // measured the same
  const int M = p.M, tm = blockIdx.x;
  const int m0 = tm * FM;

  if ((p.lda == 2048 || p.lda == 4096 || p.lda == 8192) && N <= 128 && gridDim.x > F_PLACES / 2 &&
      (int64_t)gridDim.x * (p.K / BK) >= 48 * F_PLACES && tm < F_PLACES)
    for (int i = tm / NXCD % 32; i > 0; --i) __builtin_amdgcn_s_sleep(32);   // (2048 clocks each)

  // direct loads, 1 KB each, as byte offsets of the lane from the tile's first row.  W: 8 rows x 128 bytes; lane l
  // fills slot l % 8 of row l / 8 and fetches logical chunk slot ^ f(row), f = the row bits 1, 3, 4 that vary
  // inside a (permuted) fragment.  Token rows: 16 rows x 64 bytes, contiguous; slot l % 4 of row l / 4, f = (row >> 2) & 3.
  const int first = m0 < M ? m0 : M - 1;
  uint32_t va[F_LOADS], vb[F_LOADS];
#pragma unroll
  for (int i = 0; i < F_LOADS; ++i) {
    const int r = (wave * F_LOADS + i) * 8 + (lane >> 3);
    const int row = m0 + r < M ? m0 + r : M - 1;      // (at most 127 rows of 2 MB behind `first`)
    va[i] = (uint32_t)(row - first) * (uint32_t)(p.lda * 2) + (((lane & 7) ^ (((r >> 1) & 1) | (((r >> 3) & 3) << 1))) << 4);
    const int q = (wave * F_LOADS + i) * 16 + (lane >> 2);
    vb[i] = (uint32_t)(q < N ? q : N - 1) * (FK * 2) + (((lane & 3) ^ ((q >> 2) & 3)) << 4);
  }
  const uint64_t a_base = (uint64_t)(p.A + (int64_t)first * p.lda), b_base = (uint64_t)p.B;
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + wave * (F_LOADS * 1024));
  auto load = [](uint32_t voff, uint64_t base, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(voff), "s"(base), "s"(lds) : "memory");
  };
  const int nk = p.K / FK, nc = p.K / BK;             // (nk is a multiple of 4)
  // (loads that would run past the end fetch the first chunk or stage again, into slots nobody reads)
  auto load_a = [&](int c, uint32_t slot) {
    c = c < nc ? c : c - nc;
    const uint64_t base = a_base + (uint64_t)c * (BK * 2) + (c >= p.a_tail_panel ? p.a_tail_delta : 0);
#pragma unroll
    for (int i = 0; i < F_LOADS; ++i) load(va[i], base, lds_wave + slot + i * 1024);
  };
  auto load_b = [&](int kt, uint32_t slot) {
    kt = kt < nk ? kt : kt - nk;
    const uint64_t base = b_base + (uint64_t)kt * (uint64_t)p.ldb * (FK * 2);
#pragma unroll
    for (int i = 0; i < F_LOADS; ++i) load(vb[i], base, lds_wave + slot + i * 1024);
  };

  if (wave * 64 >= N) {
    // no tokens: this wave's share of W, and the barriers
    load_a(0, 0);
    for (int c = 0; c < nc; ++c) {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
      __syncthreads();
      load_a(c + 1, (c & 1) ? 0 : F_CHUNK);
      __syncthreads();
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));        // no direct load may outlive the wave
    return;
  }

  float zt[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int n = wave * 64 + j * 16 + frow;
    zt[j] = p.zt[n < N ? n : N - 1];
  }
  const int chunk_x = ((frow >> 1) & 1) | ((frow >> 2) << 1), a_row = (8 * (frow >> 2) + (frow & 3)) * (BK * 2);
  const int a_off[2] = {a_row + ((fq ^ chunk_x) << 4), a_row + (((4 | fq) ^ chunk_x) << 4)};
  const int b_off = F_B + (wave * 64 + frow) * (FK * 2) + ((fq ^ (frow >> 2)) << 4);

  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  load_a(0, 0);
  load_b(0, F_B);
  load_b(1, F_B + F_STAGE);
  uint32_t sa = 0, sb = 0, sb_load = 2 * F_STAGE;
  auto next = [](uint32_t s) { return s == (F_STAGES - 1) * F_STAGE ? 0u : s + F_STAGE; };
  int kt = 0;
  do {                                                // (K is at least 128)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      // Stage kt + 2 is issued in step kt, chunk c + 1 before it in the first step of chunk c.  So this step's stage
      // (and chunk) have landed when what the step before issued is outstanding: a stage, or a chunk and a
      // stage.  Behind the barrier every wave's have, and every wave has read the slots that the loads refill.
      if (ks == 0) __builtin_amdgcn_s_waitcnt(waitcnt_vm(F_LOADS)); else __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * F_LOADS));
      __syncthreads();
      if (ks == 0) load_a(kt / 2 + 1, sa ^ F_CHUNK);
      load_b(kt + ks + 2, F_B + sb_load);
      const unsigned char* base_a = smem + sa + a_off[ks];
      const unsigned char* base_b = smem + sb + b_off;
      bf16x8 fb[4], fa[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(base_b + j * 1024);
#pragma unroll
      for (int i = 0; i < 8; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(base_a + (i >> 1) * 4096 + (i & 1) * 512);
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (i < 7 || j < 3) mfma16(acc[i][j], fa[i], fb[j]); else mfma16_then_wait(acc[i][j], fa[i], fb[j]);
        }
      sb = next(sb);
      sb_load = next(sb_load);
    }
    sa ^= F_CHUNK;
    kt += 2;
  } while (kt < nk);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  forward_epilogue<4>(p, acc, [&](int j) { return zt[j]; }, m0, 0, tm, 0, wave, N);
}

// ---------------------------------------------------------------------------------------------
// dW of few rows: 128 x 256 tiles (vocabulary x hidden), two workgroups per compute unit (72 KB of LDS each).
// With few rows a tile of dW is a short K loop and 256 KB of stores, and with one workgroup per compute unit neither
// overlaps the other: 28 us per 256 x 256 tile of 384 rows, 9 of them in the K loop, the stores of 2.5 GB taking 450 of
// the launch's 900 us.  Here one workgroup's products run under the other's stores.  What the loads then cost is
// L2 requests (one per clock and channel, of 64 or 128 bytes): the hidden rows lie in blocks of 32 token rows
// ([rows / 32][dp][32], written so by launch_backward_rows_b16), so that a 32-wide K step is whole lines; as rows of
// Ht, 64 bytes at a time, the launch was no faster than the large tile.  Stores are whole lines as well (lanes exchange
// 16-byte pieces so that an instruction covers 8 rows x 128 bytes) and, where rows of dW are whole lines,
// streaming: dW does not displace the operands (327 rows, d = 4096, in a loss call 957 and 748 us, 893 on the large tile; with rows that straddle lines
// streaming costs instead, 150 rows, d = 712 45 and 68).  32 consecutive tiles per XCD, whose stores then lie
// 4 MB and not 8 MB apart (400 rows, V = 140000, d = 2048 473 and 435).  Launch, us, large tile and this one:
// V = 151936, d = 4096, 150 rows 767 and 647, 400 rows 1000 and 856, 900 rows 1470 and 1340; d = 1536, 400 rows 376 and 348;
// accumulating 400 rows 1413 and 1215, 533 and 480; V = 50257, d = 712 79 and 69, accumulating 114 and 92.
// ---------------------------------------------------------------------------------------------
constexpr int DM = 128, DN = 256, DK = kRowBlock, DSTAGES = 3;
constexpr int D_A = DK * DM * 2, D_STAGE = D_A + DN * DK * 2, D_LDS = DSTAGES * D_STAGE;   // 24 KB per stage
constexpr int D_LOADS = 6;                                          // direct loads per wave and stage: 2 of A, 4 of B
// Passes of at most kFewDwRows rows: from there on the large tile's K loop, which moves half the panel bytes per product, counts
// for more than the stores.  Call with dW alone, overwriting, us, large tile and this one: d = 1024 (4 tile columns),
// V = 38405, 150 rows 125 and 105, 900 rows 229 and 209; V = 151936, 150 rows 373 and 336, 1000 rows 716 and 700; d = 2048,
// V = 38405 213 and 170, 379 and 353; V = 151936 656 and 617, 1278 and 1291; d = 3072, V = 102405, 150 rows 646 and
// 595, 900 rows 1277 and 1243; d = 4096, V = 153605 1235 and 1140, 2427 and 2364; accumulating launches gain as much or more; 1536
// rows 0.92 - 1.05.  The other way up to there: V = 128256, d = 1024, behind a dH launch, whose 7.8 rounds of large
// tiles leave little to gain, 327 rows 483 and 484, 1000 rows 825 and 846 a call.
constexpr int kFewDwRows = 1024;

__global__ __launch_bounds__(NTHREADS, 2) void dw_few_bf16(Params p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int frow = lane & 15, fq = lane >> 4, wm = wave >> 1, wn = wave & 1;
  int64_t nv64 = *p.n_scored - p.chunk_start;
  const int nvalid = nv64 < 0 ? 0 : (nv64 > p.chunk_rows ? p.chunk_rows : (int)nv64);
  if (nvalid == 0 && !p.overwrite) return;
  const int Mt = (p.V + DM - 1) / DM, Nt = (p.d + DN - 1) / DN;
  int tm, tn;
  if (!dealt_tile(blockIdx.x, Mt, Nt, tm, tn)) return;
  const int m0 = tm * DM, n0 = tn * DN;
  const int nk = dw_panels(nvalid, p.K) * (BK / DK);

  // direct loads, 1 KB each.  A, K-major: 4 k rows x 256 bytes; lane l fills chunk slot l % 16 of row l / 16 and fetches
  // logical chunk slot ^ (kswz(k) << 1).  B: 16 rows x 64 bytes, contiguous; slot l % 4 of row l / 4, swizzle (row >> 2) & 3.
  const uint16_t* src[D_LOADS];
  uint32_t dst[D_LOADS];
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
#pragma unroll
  for (int i = 0; i < D_LOADS; ++i) {
    if (i < 2) {
      const int blk = wave * 2 + i, k = blk * 4 + (lane >> 4);
      const int col = m0 + (((lane & 15) ^ (kswz(k) << 1)) << 3);
      src[i] = p.A + (int64_t)k * p.lda + (col < p.V ? col : m0);
      dst[i] = __builtin_amdgcn_readfirstlane(lds_base + blk * 1024);
    } else {
      const int blk = wave * 4 + i - 2, r = blk * 16 + (lane >> 2);
      const int n = n0 + r < p.N ? n0 + r : p.N - 1;
      src[i] = p.B + (int64_t)n * DK + (((lane & 3) ^ ((r >> 2) & 3)) << 3);
      dst[i] = __builtin_amdgcn_readfirstlane(lds_base + D_A + blk * 1024);
    }
  }
  const int64_t a_step = (int64_t)DK * p.lda * 2, b_step = p.ldb * (DK * 2);
  auto load = [&](int kt, uint32_t stage) {
    kt = kt < nk ? kt : nk - 1;
#pragma unroll
    for (int i = 0; i < D_LOADS; ++i) {
      uint64_t addr;
      asm volatile("s_mov_b32 m0, %3\n\tv_lshl_add_u64 %0, %1, 0, %2\n\tglobal_load_lds_dwordx4 %0, off"
                   : "=&v"(addr) : "v"(src[i]), "s"(kt * (i < 2 ? a_step : b_step)), "s"(dst[i] + stage) : "memory");
    }
  };
  const int kr = 8 * fq + (frow >> 2);
  const int a_base = kr * (DM * 2) + ((kswz(kr) ^ (wm * 4)) << 5) + ((frow & 3) << 3);
  const int b_base = D_A + (wn * 128 + frow) * (DK * 2) + ((fq ^ (frow >> 2)) << 4);
  f32x4 acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (nk > 0) {
    load(0, 0);
    load(1, D_STAGE);
    uint32_t st = 0, st_load = 2 * D_STAGE;
    for (int kt = 0; kt < nk; ++kt) {
      // (as in forward_few_bf16: this stage has landed when only the next one's loads are outstanding)
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(D_LOADS));
      __syncthreads();
      load(kt + 2, st_load);
      bf16x8 fa[4], fb[8];
      const unsigned char* base = smem + st;
#pragma unroll
      for (int j = 0; j < 8; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(base + b_base + j * 16 * (DK * 2));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        typedef short v4i16 __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) v4i16* lds_v4i16;
        unsigned char* q = smem + st + (a_base ^ (i << 5));
        const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)q);
        const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(q + 4 * (DM * 2)));
        fa[i] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
      st = st == (DSTAGES - 1) * D_STAGE ? 0 : st + D_STAGE;
      st_load = st_load == (DSTAGES - 1) * D_STAGE ? 0 : st_load + D_STAGE;
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));        // no direct load may outlive the wave
  }
  // The accumulators hold, per lane, row m0 + wm * 64 + i * 16 + frow, columns n0 + wn * 128 + j * 16 + 4 fq + e.  Of blocks j
  // and j + 1, lanes frow < 8 and frow >= 8 exchange halves: the first of a pair of stores takes rows 0 - 7 and 32
  // columns, the second rows 8 - 15.
  const int v0 = m0 + wm * 64 + (frow & 7), nb = n0 + wn * 128 + 16 * (frow >> 3) + 4 * fq;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    f32x4 x[8], old[8];
    float* at[8];
    bool ok[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int v = v0 + i * 16 + 8 * (j & 1), n = nb + 16 * (j & ~1);
      ok[j] = v < p.V && n < p.d;
      at[j] = p.dW + (int64_t)v * p.d + n;
      const f32x4 a = acc[i][j & ~1], b = acc[i][j | 1];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ia = __float_as_int(a[e]), ib = __float_as_int(b[e]);
        x[j][e] = __int_as_float((j & 1) == 0 ? __builtin_amdgcn_update_dpp(ia, ib, 0x128, 0xf, 0xc, false)
                                              : __builtin_amdgcn_update_dpp(ib, ia, 0x128, 0xf, 0x3, false));
      }
    }
    if (!p.overwrite) {
#pragma unroll
      for (int j = 0; j < 8; ++j) if (ok[j]) old[j] = *reinterpret_cast<const f32x4_any*>(at[j]);
#pragma unroll
      for (int j = 0; j < 8; ++j) if (ok[j]) x[j] = old[j] + x[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (ok[j]) {
        if (p.streaming) asm volatile("global_store_dwordx4 %0, %1, off nt\n\ts_nop 1" :: "v"(at[j]), "v"(x[j]) : "memory");
        else *reinterpret_cast<f32x4_any*>(at[j]) = x[j];
      }
  }
}

// dW tail.  The workgroup -> tile mapping runs whole super-tile rows of sup_m tile rows; V / 256
// tile rows leave a last, ragged super-tile row (2 tile rows x 16 tiles at V = 151936, d = 4096)
// that keeps an eighth of the compute units busy for the time of a full tile while the others
// idle: 2.3 % of the launch.  Those tiles can be cut into up to 8 slices of the contraction (the
// pass's token rows), work items a fraction of a tile long that fill the compute units the whole
// tiles leave idle at the end.  The slices store their accumulators to a scratch area and
// dw_tail_reduce adds them, slice 0 first, into dW: the result does not depend on execution order.
// Workgroup b runs on XCD b % 8 whatever else is free, so the plan is made per XCD: a model of
// the launch (32 compute units per XCD, whole tiles in id order, then the items, each on the compute unit
// that is free first) gives the time the last item ends for every split and for the unsplit mapping; the
// best one is taken, and the items are dealt to the XCDs as the model placed them.  Host code of every
// dW launch: an XCD's compute units are free at two times only (those with and without one whole tile
// more), so the model keeps two groups of them per XCD and fills a group at a time.  With every compute unit
// on its own, and compiled without optimisation, the plan took 680 us of host time at V = 151936, d = 4096
// and 490 at V = 32000, d = 2048 (where the launch takes 110 us); now 3 and 1.
struct DwTailPlan { int m0, rows, split, first[NXCD + 1]; };
DwTailPlan dw_tail_plan(int Mt, int Nt, int sup_m, int sup_n) {
  constexpr double kItemOverhead = 0.02;         // prologue, partial-tile store, reduce: in tile times
  DwTailPlan best = {Mt / sup_m * sup_m, Mt % sup_m, 0, {}};
  const int tiles = best.rows * Nt;
  if (tiles == 0 || best.m0 == 0) return best;
  const int sNt = (Nt + sup_n - 1) / sup_n;
  // tiles per XCD of the first `rows_m` tile rows under the super-tile mapping
  auto tiles_per_xcd = [&](int rows_m, int (&t)[NXCD]) {
    for (int x = 0; x < NXCD; ++x) t[x] = 0;
    const int sMt = (rows_m + sup_m - 1) / sup_m;
    for (int s = 0; s < sMt * sNt; ++s) {
      const int rm = rows_m - (s / sNt) * sup_m, rn = Nt - (s % sNt) * sup_n;
      t[s % NXCD] += (rm < sup_m ? rm : sup_m) * (rn < sup_n ? rn : sup_n);
    }
  };
  int t_all[NXCD], t_main[NXCD];
  tiles_per_xcd(Mt, t_all);
  tiles_per_xcd(best.m0, t_main);
  double unsplit = 0, whole_end = 0;
  for (int x = 0; x < NXCD; ++x) {
    const double all = (t_all[x] + kXcdCus - 1) / kXcdCus, main = (t_main[x] + kXcdCus - 1) / kXcdCus;
    unsplit = all > unsplit ? all : unsplit;
    whole_end = main > whole_end ? main : whole_end;
  }
  double best_end = unsplit - kItemOverhead;     // a split has to beat the plain mapping by a margin
  for (int split = 2; split <= 8 && tiles * split <= kDwTailMaxItems; ++split) {
    struct Group { double free_at; int units, left; };   // `left` of the units have not taken an item at this time yet
    Group group[2 * NXCD];
    for (int x = 0; x < NXCD; ++x) {
      const int more = t_main[x] % kXcdCus;
      const double base = t_main[x] / kXcdCus;
      group[2 * x] = {base, kXcdCus - more, kXcdCus - more};
      group[2 * x + 1] = {base + 1, more, more};
    }
    int count[NXCD] = {};
    double end = whole_end;
    for (int items = tiles * split; items > 0;) {
      int f = 0;                                 // free first (units - more is at least 1: group 0 is never empty)
      for (int i = 1; i < 2 * NXCD; ++i)
        if (group[i].units > 0 && group[i].free_at < group[f].free_at) f = i;
      const int n = items < group[f].left ? items : group[f].left;
      const double ends = group[f].free_at + (1.0 / split + kItemOverhead);
      end = ends > end ? ends : end;
      count[f / 2] += n;
      items -= n;
      group[f].left -= n;
      if (group[f].left == 0) { group[f].free_at = ends; group[f].left = group[f].units; }
    }
    if (end < best_end - 1e-9) {
      best_end = end; best.split = split; best.first[0] = 0;
      for (int x = 0; x < NXCD; ++x) best.first[x + 1] = best.first[x] + count[x];
    }
  }
  return best;
}

__global__ __launch_bounds__(256) void dw_tail_reduce(const float* __restrict__ part, int tiles, int split, int Nt,
                                                      int tail_m0, int V, int d, float* __restrict__ dW,
                                                      int overwrite, const int64_t* __restrict__ n_scored,
                                                      int64_t chunk_start, int chunk_rows) {
  int64_t nv64 = *n_scored - chunk_start;
  const int nvalid = nv64 < 0 ? 0 : (nv64 > chunk_rows ? chunk_rows : (int)nv64);
  if (!overwrite && nvalid == 0) return;              // the GEMM launch left dW (and part) alone
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int t = (int)(q / (BM * BN)), within = (int)(q % (BM * BN));
  if (t >= tiles) return;
  const int v = (tail_m0 + t / Nt) * BM + within / BN, n = (t % Nt) * BN + within % BN;
  if (v >= V || n >= d) return;
  float s = 0.f;
  const int slices = slices_in_use(dw_panels(nvalid, chunk_rows), split);
  for (int k = 0; k < slices; ++k) s += part[((int64_t)k * tiles + t) * (BM * BN) + within];
  float* out = dW + (int64_t)v * d + n;
  *out = overwrite ? s : *out + s;
}

// Adds the slices of the dH launch's tail tiles (slice 0 first), applies the row scale and scatters
// the rows to their slots: 8 columns per thread.  Blocks beyond the tiles that the device finds cut
// return at once.
__global__ __launch_bounds__(256) void dh_tail_reduce(Params p) {
  int64_t nv64 = *p.n_scored - p.chunk_start;
  const int M = nv64 < 0 ? 0 : (nv64 > p.chunk_rows ? p.chunk_rows : (int)nv64);
  const int Mt = (M + BM - 1) / BM, Nt = (p.N + BN - 1) / BN;
  const int tiles = Mt * Nt, whole = tiles / kRound * kRound, rest = tiles - whole;
  const int t = blockIdx.x / (BM * BN / 2048);
  if (t >= rest) return;
  const int split = dh_split(rest, p.K / BK, p.max_items);
  if (split == 1) return;
  int tm, tn;
  tile_at(whole + t, Mt, Nt, tm, tn);
  const int within = (blockIdx.x % (BM * BN / 2048)) * 2048 + threadIdx.x * 8;
  const int m = tm * BM + within / BN, n = tn * BN + within % BN;
  if (m >= M || n >= p.d) return;
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll 4
  for (int s = 0; s < split; ++s) {
    const f32x4* q = reinterpret_cast<const f32x4*>(p.tail_part + ((int64_t)s * rest + t) * (BM * BN) + within);
    lo += q[0];
    hi += q[1];
  }
  const float sc = p.row_scale[m];
  const int64_t at = (int64_t)p.row_index[m] * p.d + n;
  if (p.dh_f32) {
    float* out = static_cast<float*>(p.dH) + at;
#pragma unroll
    for (int e = 0; e < 4; ++e) { out[e] = sc * lo[e]; out[4 + e] = sc * hi[e]; }
  } else {
    bf16x8 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) { h[e] = (__bf16)(sc * lo[e]); h[4 + e] = (__bf16)(sc * hi[e]); }
    *reinterpret_cast<bf16x8*>(static_cast<uint16_t*>(p.dH) + at) = h;
  }
}

template <int MODE>
void launch(Params& p, hipStream_t stream) {
  static LdsLimit lds_limit;
  lds_limit.ensure(reinterpret_cast<const void*>(&gemm_nt_bf16<MODE>), lds_bytes<MODE>());
  const int Mt = (p.M + BM - 1) / BM, Nt = (p.N + BN - 1) / BN;
  const SuperTile st = pick_super_tile(Nt);
  p.sup_m = st.m; p.sup_n = st.n;
  int blocks = MODE == MODE_DW ? num_blocks(Mt, Nt, st.m, st.n) : (Mt * Nt + NXCD - 1) / NXCD * NXCD;
  DwTailPlan tail = {0, 0, 0, {}};
  if (MODE == MODE_DW && p.tail_part != nullptr) tail = dw_tail_plan(Mt, Nt, st.m, st.n);
  if (tail.split > 0) {
    p.main_blocks = num_blocks(tail.m0, Nt, st.m, st.n);
    p.tail_m0 = tail.m0; p.tail_rows = tail.rows; p.tail_split = tail.split;
    int most = 0;
    for (int x = 0; x < NXCD; ++x) {
      p.tail_first[x] = tail.first[x];
      most = tail.first[x + 1] - tail.first[x] > most ? tail.first[x + 1] - tail.first[x] : most;
    }
    p.tail_first[NXCD] = tail.first[NXCD];
    blocks = p.main_blocks + most * NXCD;
  }
  if (MODE == MODE_DH) blocks = (Mt * Nt) / kRound * kRound + (int)round_up(dh_most_items(Mt * Nt, p.K / BK, p.max_items), NXCD);
  hipLaunchKernelGGL(gemm_nt_bf16<MODE>, dim3(blocks), dim3(NTHREADS), lds_bytes<MODE>(), stream, p);
  if (tail.split > 0) {
    const int tiles = tail.rows * Nt;
    hipLaunchKernelGGL(dw_tail_reduce, dim3(tiles * (BM * BN / 256)), dim3(256), 0, stream, p.tail_part, tiles,
                       tail.split, Nt, tail.m0, p.V, p.d, p.dW, p.overwrite, p.n_scored, p.chunk_start,
                       p.chunk_rows);
  }
  if (MODE == MODE_DH && dh_most_split(p.K / BK) > 1) {
    const int most = Mt * Nt < kRound ? Mt * Nt : kRound - 1;
    hipLaunchKernelGGL(dh_tail_reduce, dim3(most * (BM * BN / 2048)), dim3(256), 0, stream, p);
  }
}

}  // namespace

void launch_gemm_fwd_bf16(const void* W, int64_t ldw, const void* W_tail, const void* Hc, int64_t ldh, int k_len, const float* zt,
                          const int64_t* n_scored, int64_t chunk_start, int chunk_rows,
                          int V, int d, float* part_sum, float* part_ez,
                          int64_t part_stride, void* estash, int64_t lde, bool in_blocks, hipStream_t stream) {
  Params p = {};
  p.A = static_cast<const uint16_t*>(W); p.lda = ldw; p.M = V;
  p.B = static_cast<const uint16_t*>(Hc); p.ldb = ldh; p.N = chunk_rows;
  p.K = k_len;
  p.a_tail_panel = k_len / BK;                        // none
  if (W_tail != nullptr) {
    p.a_tail_panel = k_len / BK - 2;
    p.a_tail_delta = (int64_t)(reinterpret_cast<uintptr_t>(W_tail) - reinterpret_cast<uintptr_t>(W)) - (int64_t)p.a_tail_panel * (BK * 2);
  }
  p.n_scored = n_scored; p.chunk_start = chunk_start; p.chunk_rows = chunk_rows;
  p.zt = zt + chunk_start;
  p.part_sum = part_sum; p.part_ez = part_ez; p.part_stride = part_stride;
  p.estash = static_cast<uint16_t*>(estash); p.lde = lde; p.V = V; p.d = d;
  if (in_blocks) {
    static LdsLimit lds_limit;
    lds_limit.ensure(reinterpret_cast<const void*>(&forward_few_bf16), F_LDS);
    const int Mt = 2 * ((p.M + BM - 1) / BM);
    hipLaunchKernelGGL(forward_few_bf16, dim3(Mt), dim3(NTHREADS), F_LDS, stream, p);
    return;
  }
  launch<MODE_FWD>(p, stream);
}

void launch_gemm_dh_bf16(const void* E, int64_t lde, const void* W, int64_t ldw, int V,
                         const int32_t* row_index, const float* row_scale, const int64_t* n_scored,
                         int64_t chunk_start, int chunk_rows, int d, void* dH, int dh_f32,
                         float* tail_part, int tail_items, hipStream_t stream) {
  Params p = {};
  p.A = static_cast<const uint16_t*>(E); p.lda = lde; p.M = chunk_rows;
  p.row_scale = row_scale + chunk_start;
  p.B = static_cast<const uint16_t*>(W); p.ldb = ldw; p.N = d;
  p.K = (int)round_up(V, 2 * BK);
  p.row_index = row_index + chunk_start;
  p.n_scored = n_scored; p.chunk_start = chunk_start; p.chunk_rows = chunk_rows;
  p.dH = dH; p.dh_f32 = dh_f32; p.d = d; p.V = V;
  p.tail_part = tail_part; p.max_items = tail_items;
  launch<MODE_DH>(p, stream);
}

size_t gemm_tail_tile_bytes() { return (size_t)BM * BN * sizeof(float); }
int gemm_dw_tail_items() { return kDwTailMaxItems; }
bool dw_rows_in_blocks(int rows) { return rows <= kFewDwRows; }

void launch_gemm_dw_bf16(const void* E, int64_t lde, const void* Ht, int64_t ldht,
                         const int64_t* n_scored, int64_t chunk_start, int chunk_rows,
                         int V, int d, float* dW, int overwrite, float* tail_part, bool in_blocks, hipStream_t stream) {
  Params p = {};
  p.A = static_cast<const uint16_t*>(E); p.lda = lde; p.M = (int)round_up(V, kTile);
  p.B = static_cast<const uint16_t*>(Ht); p.ldb = ldht; p.N = d;
  p.K = chunk_rows;
  p.n_scored = n_scored; p.chunk_start = chunk_start; p.chunk_rows = chunk_rows;
  p.dW = dW; p.overwrite = overwrite; p.V = V; p.d = d;
  p.tail_part = tail_part;
  if (in_blocks) {
    p.N = (int)ldht;                                  // (rows of a block: d rounded up to 128)
    p.streaming = d % 32 == 0 && (reinterpret_cast<uintptr_t>(dW) & 127) == 0;
    static LdsLimit lds_limit;
    lds_limit.ensure(reinterpret_cast<const void*>(&dw_few_bf16), D_LDS);
    const int64_t tiles = (int64_t)((V + DM - 1) / DM) * ((d + DN - 1) / DN);
    hipLaunchKernelGGL(dw_few_bf16, dim3((unsigned)round_up(tiles, NXCD)), dim3(NTHREADS), D_LDS, stream, p);
    return;
  }
  launch<MODE_DW>(p, stream);
}

}  // namespace mrl

extern "C" int mrl_diag_dh_split(int32_t tail_tiles, int32_t panels, int32_t max_items) {
  using namespace mrl;
  if (tail_tiles <= 0 || tail_tiles >= kRound || panels <= 0 || max_items < tail_tiles) return MRL_ERR_SHAPE;
  return dh_split(tail_tiles, panels, max_items);
}

extern "C" int mrl_diag_dw_few_rows(void) { return mrl::kFewDwRows; }

extern "C" int mrl_diag_dw_tail_plan(int32_t V, int32_t d, int32_t* out12) {
  using namespace mrl;
  if (out12 == nullptr) return MRL_ERR_NULL;
  if (V <= 0 || d <= 0) return MRL_ERR_SHAPE;
  const int Mt = (int)(round_up(V, kTile) / BM), Nt = (d + BN - 1) / BN;
  const SuperTile st = pick_super_tile(Nt);
  const DwTailPlan t = dw_tail_plan(Mt, Nt, st.m, st.n);
  out12[0] = t.m0; out12[1] = t.rows; out12[2] = t.split;
  for (int x = 0; x <= NXCD; ++x) out12[3 + x] = t.split > 0 ? t.first[x] : 0;
  return MRL_OK;
}
