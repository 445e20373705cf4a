// bf16 MFMA tile GEMM for gfx950 with three fused epilogues.
//
// One kernel body computes C[m][n] = sum_k A[m][k] * B[n][k] for a 384 x 256 tile per workgroup: four wave64 wavefronts in a
// 2 x 2 grid, each owning a 192 x 128 sub-tile as 12 x 8 MFMA 16x16x32 accumulators (384 accumulator registers per lane, 256 of them
// in the accumulation file).  What bounds these launches is the power limit, which the chip is at with random mantissas, and the issue
// of moving operands, which leaves the matrix cores idle: a tile that moves fewer bytes per product keeps them busier, and the limit
// takes a part of that back through the clock.
// 384 x 256 is the largest tile that fits registers and LDS (two panels of 80 KB); per product it takes 17 % less from the L2
// and from LDS than 256 x 256.  Launches of 15360 rows, V = 151936, d = 4096, 256 x 256 and now, us: forward with the stash 12660 and
// 12340, dH 12740 and 11750, dW 13010 and 12080 (matrix cores busy 74 and 75, 77 and 83, 75 and 80 % of the cycles; clock 1.88 and 1.86,
// 1.84 and 1.78, 1.86 and 1.79 GHz);
// 28672 rows, V = 128256, d = 2048 11055 and 10680, 10080 and 9420, 9905 and 9000.
// The 16x16x32 shape is chosen over 32x32x16 for energy: an MFMA-only loop sustains about 13 % more FLOP/s with it.  Operand
// panels of 64 K-elements go from global memory straight into LDS (buffer_load ... lds, no staging registers)
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

#include <cstring>

namespace mrl {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // 16-byte access, 4-byte alignment

constexpr int BK = 64;
constexpr int NTHREADS = 256;
constexpr int kDwTailMaxItems = 256;                // K slices of dW tail tiles per launch: one per compute unit

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
  uint64_t cuts[4];           // FWD, DH: how the token rows are cut into tiles, two bits per 128 of them (see Cut)
  // DH
  const float* row_scale; void* dH; int dh_f32; int d; int max_items;   // max_items: partial tiles tail_part holds
  // DW
  float* dW; int overwrite; int streaming; int wide;
  // DW, K-split tail (see dw_tail_plan): workgroups from main_blocks on take the tiles of the
  // tile rows tail_m0 .. tail_m0 + tail_rows - 1, each cut into tail_split slices of the
  // contraction, and store their accumulators to tail_part instead of dW
  int main_blocks, tail_m0, tail_rows, tail_split; float* tail_part;
  int tail_first[NXCD + 1];   // items tail_first[x] .. tail_first[x + 1] - 1 run on XCD x
};

// Workgroup -> tile mapping of the launches.  Workgroups are dealt round-robin to the
// 8 XCDs, each with its own L2 and 32 compute units; 32 consecutive workgroups of one XCD take 32
// consecutive tiles, numbered down the columns of bands of tile rows, so that they share operand panels in that L2 and all XCDs
// walk the same A rows at the same time.  Bands of 8 rows of 256 in the forward (8 x 4 tiles, the tokens' side of 384) and in dH without tiles of 384, of 4
// rows of 384 in dH and dW (4 x 8): either takes 3584 rows of panels per group, the other shape 4096 (dH of 15360 rows, d = 4096 12920 and 12775 us).  The numbering runs over the VALID tiles (the scored rows are counted on the device) without
// holes: numbering super-tiles over the launch's upper bound gave each XCD fixed tile columns, and
// with 20 of 32 tile columns valid three XCDs had nothing to do (scoring 5120 of 8192 slots,
// V = 128256, d = 2048: 3233 us a call against 2088 us now).  The tiles of the last, incomplete round
// of 256 are dealt evenly.
constexpr int kXcdCus = 32;
constexpr int kRound = NXCD * kXcdCus;
__device__ __forceinline__ void tile_at(int band, int t, int Mt, int Nt, int& tm, int& tn) {
  const int first = t / (band * Nt) * band, in_band = t - first * Nt;
  const int rows = Mt - first < band ? Mt - first : band;
  tn = in_band / rows;
  tm = first + in_band - tn * rows;
}
__device__ __forceinline__ bool dealt_tile(int band, int bid, int Mt, int Nt, int& tm, int& tn) {
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
  tile_at(band, t, Mt, Nt, tm, tn);
  return true;
}

// dH: the tiles of the last, incomplete round of 256 (all of them, when a pass has few rows) are cut
// into slices of the contraction over the vocabulary, one work item each, which store their
// accumulators to a scratch area; dh_tail_reduce adds them in slice order.  A dH tile is long (2374
// panels at V = 151936, about 3.6 ms), so an idle compute unit in that round costs more than
// writing and adding the partial tiles (384 KB per item): 327 rows at d = 4096 are 16 tiles.
// The slice count is the one whose rounds of items end earliest, 1 / kItemCostInv of a tile covering an item's
// prologue, partial store and share of the reduce.  In whole numbers: the launch and the reduction each work
// it out on the device and have to come to the same answer.  Measured when it was introduced, on tiles of 256 x 256 (launch and reduce,
// V = 151936; before: whole tiles and a transposed copy of W in front): 327 rows, d = 4096, 32 tiles: 3480 -> 527 us (353 on tiles
// of 384); 5120 rows, d = 1536, 120 tiles: 3251 -> 1720 us; 47360 rows, d = 3584, 2590 tiles: 39.1 -> 35.9 ms.
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
  const int rest = tiles < kRound ? tiles : kRound - 1, n = rest * dh_most_split(panels);
  return n < max_items ? n : max_items > rest ? max_items : rest;
}
// panels per slice: an even number (the K loop's body is two panels)
__host__ __device__ inline int slice_panels(int panels, int split) { return ((panels + split - 1) / split + 1) & ~1; }
// slices that have any panels: the dW plan does not know the scored rows, and 6 panels make three slices of the
// planned 8.  (No panels at all: the first slice stores the zeros of an overwriting launch.)
__device__ inline int slices_in_use(int panels, int split) {
  const int per = slice_panels(panels, split);
  return panels > 0 ? (panels + per - 1) / per : 1;
}
// dW on 384 x 256 tiles: the same for its last round.  The contraction is as long as the pass (16 panels are 1024 rows), so an
// item's share beyond its panels counts in panels: about 6 for its prologue and its store, 12 for the launch that adds the slices.
__host__ __device__ inline int dw_split(int tail_tiles, int panels, int max_items) {
  int best = 1, end = panels + 6;
  for (int s = 2; s <= 64 && s * 8 <= panels && s * tail_tiles <= max_items; ++s) {
    const int e = (tail_tiles * s + kRound - 1) / kRound * ((panels + s - 1) / s + 6) + 12;
    if (e < end) { end = e; best = s; }
  }
  return best;
}
struct DhSplit { __device__ int operator()(int tiles, int panels, int max_items) const { return dh_split(tiles, panels, max_items); } };
struct DwSplit { __device__ int operator()(int tiles, int panels, int max_items) const { return dw_split(tiles, panels, max_items); } };
// Workgroup -> tile or slice of one, for a launch whose last round may be cut.  Returns the item's number (its place in the
// scratch area) for a slice, panels k_first .. k_first + nk - 1 of its tile; -1 for a whole tile; -2 for nothing.
template <class Split>
__device__ __forceinline__ int split_tile(int band, int bid, int Mt, int Nt, int panels, int max_items, Split split_of, int& tm, int& tn, int& k_first, int& nk) {
  const int tiles = Mt * Nt, whole = tiles / kRound * kRound, rest = tiles - whole;
  if (bid >= whole && rest > 0) {
    const int split = split_of(rest, panels, max_items);
    if (split > 1) {
      // an XCD takes consecutive items, i.e. mostly tiles of one slice
      const int items = rest * split, per = (items + NXCD - 1) / NXCD;
      const int e = bid - whole, item = e % NXCD * per + e / NXCD;
      if (e / NXCD >= per || item >= items) return -2;
      const int slice = item / rest, per_slice = slice_panels(panels, split);
      tile_at(band, whole + item - slice * rest, Mt, Nt, tm, tn);
      k_first = slice * per_slice;
      nk = panels - k_first < per_slice ? panels - k_first : per_slice;
      return item;
    }
  }
  return dealt_tile(band, bid, Mt, Nt, tm, tn) ? -1 : -2;
}
// panels of the dW contraction: the pass's valid rows, rounded up to panel pairs
__host__ __device__ inline int dw_panels(int nvalid, int chunk_rows) {
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
__device__ inline bool tile_coords(int bid, int Mt, int Nt, int sup_m, int sup_n, int& tm, int& tn) {
  const int sNt = (Nt + sup_n - 1) / sup_n, sMt = (Mt + sup_m - 1) / sup_m;
  const int xcd = bid % NXCD, local = bid / NXCD;
  const int q = local / (sup_m * sup_n), within = local % (sup_m * sup_n);
  const int s = q * NXCD + xcd;
  if (s >= sMt * sNt) return false;
  tm = (s / sNt) * sup_m + within % sup_m;
  tn = (s % sNt) * sup_n + within / sup_m;
  return tm < Mt && tn < Nt;
}

// swizzle of the K-major A panel: rows k, k+1, k+2, k+3 and k+8 (or k+16) get distinct values
__device__ inline int kswz(int k) { return (k & 3) | ((((k >> 3) ^ (k >> 4)) & 1) << 2); }

__device__ inline float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// The MFMA is issued through inline assembly with the accumulator tied in place in an
// accumulation register: left to the register allocator, a few of the 64 accumulator tuples
// that fill the accumulation file completely end up rotating through copies every iteration.
// The K loop issues the two 32-wide K steps of an accumulator back to back: the second MFMA reads
// as SrcC the register tuple the first one writes as vDst.  That dependent pair with identical
// SrcC / vDst is the case the hardware interlocks by itself (no software wait states required);
// no other instruction touches an accumulator inside the loop.  The first ordinary reads after
// the K loop come behind wait states (the compiler's hazard checker does not look into inline assembly).
__device__ __forceinline__ void mfma16(f32x4& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
// The last MFMA of a loop body whose accumulators the compiler may move behind the loop (it does, where
// paths meet): the wait states before an ordinary read of the result are part of it.
__device__ __forceinline__ void mfma16_then_wait(f32x4& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0\n\ts_nop 15\n\ts_nop 3" : "+a"(c) : "v"(a), "v"(b));
}
// The same with the accumulator in an ordinary register: the last third of a whole tile's, which do not fit the accumulation file.
__device__ __forceinline__ void mfma16_v(f32x4& c, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// An accumulation register, read where its value is used: left to the compiler, the copies out of the accumulation
// registers are hoisted to the top of the epilogue and fill the register file.
__device__ __forceinline__ float acc_now(const float& x) {
  float z;
  asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(z) : "a"(x));
  return z;
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

// Forward epilogue of a wave's 128 x (16 NJ) sub-tile: vocabulary ids from v0, token columns from n0, partial sums with
// index pidx; target_logit(j): that of the lane's token in column block j; accumulator element (i, j, e) of a lane is
// vocabulary id vrow(i, e), token column ncol_base + 16 j.
template <int NJ, class Acc, class Zt>
__device__ __forceinline__ void forward_epilogue(const Params& p, Acc read_acc, Zt target_logit, int v0, int n0, int pidx, int N) {
  const int lane = lane_now(), frow = lane & 15, fq = lane >> 4;
  const int ncol_base = n0 + frow;
      // rows = vocabulary ids, cols = token rows of the chunk.  Exponentials are taken relative to
      // the row's offset c2 = z_target * log2(e) + margin (log2 domain), one offset for all
      // vocabulary tiles of a row: e = 2^(z log2(e) - c2), clamped so that neither e nor any sum of
      // it can overflow.  The sums over the wave's 128 vocabulary ids are this tile's partials; e
      // itself, as bf16, is the backward pass's operand (dz = (-g / S)(e - S onehot)).
      constexpr float LOG2E = 1.4426950408889634f;
      const bool full = (v0 + 128 <= p.V);
          // vocabulary id of accumulator (i, e) of this lane
      auto vrow = [&](int i, int e) {
        return v0 + 32 * (i >> 1) + 8 * fq + 4 * (i & 1) + e;
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
          uint16_t* erow = p.estash + (int64_t)n * p.lde + v0 + 8 * fq;
          float s = 0.f, t = 0.f;
  #pragma unroll
          for (int q = 0; q < 4; ++q) {
            // accumulators 2q and 2q+1 hold 8 consecutive vocabulary ids of this lane
            bf16x8 h;
  #pragma unroll
            for (int u = 0; u < 2; ++u)
  #pragma unroll
              for (int e = 0; e < 4; ++e) {
                const float z = read_acc(2 * q + u, j, e);
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
// The tile.  Per wave 8 blocks of 16 on the resident side (256 of the tile), NJ on the ring side (32 NJ: 384, or 128 in dH).  The forward has
// the vocabulary on the resident side and the tokens in the ring, dH the hidden columns and the tokens, dW the hidden columns and
// the vocabulary: the ring side is the one that is cut into tiles of other sizes.
// ---------------------------------------------------------------------------------------------
constexpr int RES = 256;                              // resident side of a tile
constexpr int kWide = 12;                             // ring blocks per wave of a whole tile
constexpr int RING = 32 * kWide;                      // ring side of a whole tile: 384
template <int NJ> constexpr int wave_bytes() { return (8 + NJ) * 1024; }     // of a slot: what one wave loads
template <int NJ> constexpr int tile_slots() { return NJ == 4 ? 3 : 2; }
template <int NJ> constexpr int tile_lds() { return tile_slots<NJ>() * 4 * wave_bytes<NJ>(); }
constexpr int DHSTAGE_LD = 128 + 8;                   // bf16 elements per row of the dH epilogue's staging area
static_assert(tile_lds<12>() == 160 * 1024 && tile_lds<4>() <= tile_lds<12>(), "all of a compute unit's LDS");
static_assert(4 * 96 * DHSTAGE_LD * 2 <= tile_lds<12>(), "half a wave's rows, four waves");

// The kernel's arguments, read again where they are used: kept alive across the forward's K loop they cost scalar registers (15360 rows,
// d = 2048 5556 us a scoring call, 5673 without); dH and dW have enough (5120 rows, d = 1536 dH 1553 and 1535 us, dW 1688 and 1667).
__device__ __forceinline__ const Params& args_now() {
  typedef const __attribute__((address_space(4))) Params* KernArg;
  KernArg arg = (KernArg)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(arg));
  return *(const Params*)arg;
}

// Ring block i of half wr of a K-major ring panel (dW): its first row within the tile.  The first eight of a half are one 256-byte group
// of a panel row, and the swizzle stays within such groups.
__device__ __forceinline__ int ring_kmajor_row(int i, int wr) { return i < 8 ? wr * 128 + i * 16 : 256 + wr * 64 + (i - 8) * 16; }

// dH epilogue of a wave's (16 NJ) x 128 sub-tile: token rows from m0, hidden columns from n0 (from tm0, tn0 within the tile), M valid rows.
// Rows of the stash times W are the rows' dz W up to their scale -g / S, applied here.
template <int NJ, class Acc>
__device__ __forceinline__ void dh_epilogue(const Params& p, unsigned char* smem, Acc read_acc, int wave, int m0, int tm0, int n0, int tn0,
                                            int M, float* tail_out) {
  const int lane = lane_now(), frow = lane & 15, fq = lane >> 4;
  if (tail_out != nullptr) {
    // a slice of the contraction: the accumulators as they are, rows of 256
#pragma unroll
    for (int i = 0; i < NJ; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float* row = tail_out + (tm0 + i * 16 + 4 * fq + e) * RES + tn0 + frow;
#pragma unroll
        for (int j = 0; j < 8; ++j) row[j * 16] = read_acc(i, j, e);
      }
    return;
  }
  if (p.dh_f32) {
#pragma unroll
    for (int i = 0; i < NJ; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + i * 16 + 4 * fq + e;
        if (m < M) {
          const float sc = p.row_scale[m];
          float* row = reinterpret_cast<float*>(p.dH) + (int64_t)p.row_index[m] * p.d;
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const int n = n0 + j * 16 + frow;
            const float x = read_acc(i, j, e);
            if (n < p.d) row[n] = sc * x;
          }
        }
      }
    return;
  }
  // The wave's rows as bf16 through its own part of LDS, half of them at a time, then 16 lanes store 256 bytes of a row.
  __syncthreads();                                    // (the panels are not read any more, and no wave's loads are outstanding)
  __bf16* const st = reinterpret_cast<__bf16*>(smem) + wave * (8 * NJ * DHSTAGE_LD);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
#pragma unroll
    for (int i = 0; i < NJ / 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = i * 16 + 4 * fq + e, m = m0 + half * (8 * NJ) + r;
        const float sc = p.row_scale[m < M ? m : M - 1];
#pragma unroll
        for (int j = 0; j < 8; ++j) st[r * DHSTAGE_LD + j * 16 + frow] = (__bf16)(sc * read_acc(half * (NJ / 2) + i, j, e));
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 4
    for (int k = 0; k < 2 * NJ; ++k) {
      const int r = k * 4 + fq, m = m0 + half * (8 * NJ) + r, n = n0 + frow * 8;
      if (m < M && n < p.d) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(&st[r * DHSTAGE_LD + frow * 8]);
        *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(p.dH) + (int64_t)p.row_index[m] * p.d + n) = v;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// dW epilogue: vocabulary rows from m0 up to v_end on the ring side, hidden columns from n0; fp32 accumulate into dW.  With the MFMA's operands
// swapped a lane holds four consecutive columns of a row, so that dW is read and written 16 bytes at a time (d is a multiple
// of 8; with 4-byte accesses the launch took 1128 instead of 1023 us for 512 rows, V = 151936, d = 4096, and 127 instead
// of 109 for V = 32000, d = 2048).  The old values of a 16-row band are fetched as a batch before any store, so
// that their latencies overlap.  A K slice of a tail tile stores its partial tile as it is, rows of 256, to the scratch
// area instead (dw_wide_reduce or, of 256 x 256 tiles, dw_tail_reduce adds the slices in their order): the same code with the tile's own origin, row stride and bounds.
template <int NJ>
__device__ __forceinline__ void dw_epilogue(const Params& p, f32x4 (&acc)[NJ][8], int wr, int m0, int n0, int res0, int v_last, float* tail_out) {
  const int lane = lane_now(), frow = lane & 15, fq = lane >> 4;
  const bool tail = tail_out != nullptr;
  float* const dst = tail ? tail_out : p.dW;
  const int64_t ld = tail ? RES : p.d;
  const int v_org = tail ? m0 : 0, n_org = tail ? res0 : 0;
  const int v_end = tail ? m0 + 32 * NJ : v_last, n_end = tail ? res0 + RES : p.d;
  const bool overwrite = tail || p.overwrite;
  const int nbase = n0 + 4 * fq;
#pragma unroll
  for (int i = 0; i < NJ; ++i) {
    const int v = m0 + ring_kmajor_row(i, wr) + frow;
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

// one direct load of 1 KB to LDS address slot + lds, from byte voff + soff behind the descriptor's base
__device__ __forceinline__ void load_lds16(uint32_t voff, uint32_t soff, const u32x4& desc, uint32_t slot, uint32_t lds) {
  uint32_t off;
  asm volatile("s_add_u32 m0, %4, %5\n\tv_add_u32 %0, %3, %1\n\tbuffer_load_dwordx4 %0, %2, 0 offen lds"
               : "=&v"(off) : "v"(voff), "s"(desc), "s"(soff), "s"(slot), "s"(lds) : "memory", "scc");
}

// One tile's product and epilogue: ring rows ring0 .. ring_end - 1 (at most 32 NJ) times resident block res_tile, panels
// k_first .. k_first + nk - 1.
// A panel is 16 NJ products in duos: two ring blocks times the eight resident ones, the two 32-wide K steps of an accumulator back to
// back (keeping an accumulator for two products costs about 5 % less energy than touching another one each time).  Registers:
// the resident fragments of a panel in one set, each pair read again for the next panel behind its last product in the
// panel's last duo and needed 32 products later; the ring's in two sets, a duo ahead.  384 + 64 + 32 of 512 registers.
// Side work stands between products, one piece behind each: a wave issues in order and the matrix pipe takes a product
// every 16 cycles, so what fits the 12 cycles left over is free, and a block of it idles the pipe (the advance to the next panel as
// one block behind the barrier cost 1.5 - 2 %).
//   barrier (fourth product of the last duo): the next panel has landed, and every wave's reads of this one are done
//   behind it, in the last duo: ring blocks 0 and 1 and the resident blocks of the next panel
//   from there on, every sixth product: the 8 + NJ loads of the panel behind the next, into the slot just released (15360 rows,
//   d = 4096: every third 1 % slower, every eighth 0.5 %: four waves issue together and a load takes the load path 23 cycles)
//   other duos: the next duo's ring blocks; then, in four pieces, the loads' advance by a panel
// Loads go through buffer descriptors that end with the operand's last row and are emptied behind the last panel: edges need
// no clamped addresses, and nothing is fetched twice at a tile's end.
template <int MODE, int NJ>
__device__ __forceinline__ void tile_product(const Params& args, unsigned char* smem, int ring_tile, int res_tile, int ring0, int ring_end,
                                             int k_first, int nk, float* tail_out) {
  constexpr bool RES_KMAJOR = MODE == MODE_DH, RING_KMAJOR = MODE == MODE_DW;
  constexpr int ND = NJ / 2, kLoads = 8 + NJ, kSlots = tile_slots<NJ>(), kWave = wave_bytes<NJ>(), kSlot = 4 * kWave;
  // Places in a panel's sequence of 16 NJ products: the barrier behind which the next panel may be read and this one's slot
  // filled again, and from there the slot's loads.
  constexpr int kPanel = 16 * NJ, kBarrier = kPanel - 32 + 3, kFirst = 2, kGap = NJ == 4 ? 3 : 6;
  constexpr int kEarlyLoads = (kPanel - 1 - kBarrier - kFirst) / kGap + 1;     // those of the next slot that come before the panel's end
  static_assert(kFirst + kGap * (kLoads - 1) < kPanel - 14, "a slot's loads are issued before the next barrier");
  const Params& p = MODE == MODE_FWD ? args_now() : args;     // (see there)
  // (wave-uniform all of them; some come out of integer divisions, which run on the vector unit)
  ring_tile = __builtin_amdgcn_readfirstlane(ring_tile); res_tile = __builtin_amdgcn_readfirstlane(res_tile);
  ring0 = __builtin_amdgcn_readfirstlane(ring0); ring_end = __builtin_amdgcn_readfirstlane(ring_end);
  k_first = __builtin_amdgcn_readfirstlane(k_first); nk = __builtin_amdgcn_readfirstlane(nk);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave >> 1, ws = wave & 1, frow = lane & 15, fq = lane >> 4;
  const int res0 = res_tile * RES;
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + wave * kWave);

  // ---- direct loads
  const uint16_t* const res_ptr = MODE == MODE_FWD ? p.A : p.B;
  const uint16_t* const ring_ptr = MODE == MODE_FWD ? p.B : p.A;
  const int64_t res_ld = MODE == MODE_FWD ? p.lda : p.ldb, ring_ld = MODE == MODE_FWD ? p.ldb : p.lda;
  const uint32_t res_ld2 = (uint32_t)(res_ld * 2), ring_ld2 = (uint32_t)(ring_ld * 2);
  const int rot_res = 4 * (ring_tile & 1);
  const int rot_ring = !RING_KMAJOR ? 2 * (res_tile & 7) % NJ : 6 * (res_tile & 1);
  constexpr int kResKinds = MODE == MODE_DW ? 2 : 4, kRingKinds = !RING_KMAJOR ? 2 : 6;
  static_assert(!RING_KMAJOR || NJ == kWide, "places of a K-major ring's loads");
  uint32_t vres[kResKinds], vring[kRingKinds];
  auto chunk16 = [&](int row) { return (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) << 4); };
#pragma unroll
  for (int q = 0; q < kResKinds; ++q) {
    const int b = ((RES_KMAJOR ? (q & 1) + 4 * (q >> 1) : q) + rot_res) & 7;
    if (RES_KMAJOR) {
      vres[q] = (uint32_t)(lane >> 5) * res_ld2 + (((lane & 31) ^ (kswz(16 * wave + 2 * b + (lane >> 5)) << 1)) << 4);
    } else {
      const int r = b * 8 + (lane >> 3);
      vres[q] = (uint32_t)(lane >> 3) * res_ld2 + (MODE == MODE_FWD ? (uint32_t)(((lane & 7) ^ (((r >> 1) & 1) | (((r >> 3) & 3) << 1))) << 4) : chunk16(r));
    }
  }
#pragma unroll
  for (int q = 0; q < kRingKinds; ++q) {
    if (!RING_KMAJOR) {
      vring[q] = (uint32_t)(lane >> 3) * ring_ld2 + chunk16((q + rot_ring) * 8 + (lane >> 3));
    } else {
      const int b = (q % 3 + 6 * (q / 3) + rot_ring) % NJ;
      const int c = 64 * (b % 3) + lane, r = c / (4 * NJ), k = 4 * (b / 3) + r;
      const int col = (c % (4 * NJ)) ^ (kswz(16 * wave + k) << 1);
      // (columns from V on are not fetched: their products are not stored)
      vring[q] = ring0 + col * 8 < p.V ? (uint32_t)r * ring_ld2 + (col << 4) : 0x80000000u;
    }
  }
  uint32_t from[kLoads], to[kLoads];
#pragma unroll
  for (int l = 0; l < kLoads; ++l) {
    const int b = l < 8 ? (l + rot_res) & 7 : (l - 8 + rot_ring) % NJ;
    const uint32_t rows = l < 8 ? (RES_KMAJOR ? 2 * b : 8 * b) : (!RING_KMAJOR ? 8 * b : 4 * (b / 3));
    from[l] = __builtin_amdgcn_readfirstlane(rows * (l < 8 ? res_ld2 : ring_ld2));
    to[l] = __builtin_amdgcn_readfirstlane((l < 8 ? b : b + 8) * 1024);
  }
  auto kind = [](int l) {
    if (l < 8) return MODE == MODE_FWD ? l & 3 : MODE == MODE_DW ? l & 1 : (l & 1) | ((l >> 2) << 1);
    l -= 8;
    return !RING_KMAJOR ? l & 1 : l % 3 + 3 * (l / 6);
  };
  u32x4 dres, dring;
  auto set = [](u32x4& d, const uint16_t* at, uint32_t bytes) {
    const uint64_t a = (uint64_t)at;
    d[0] = __builtin_amdgcn_readfirstlane((uint32_t)a); d[1] = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
    d[2] = __builtin_amdgcn_readfirstlane(bytes); d[3] = 0x00020000u;
  };
  auto move = [](u32x4& d, int64_t by) {
    const uint64_t a = (((uint64_t)d[1] << 32) | d[0]) + (uint64_t)by;
    d[0] = (uint32_t)a; d[1] = (uint32_t)(a >> 32);
  };
  auto rows_of = [&](u32x4& d, const uint16_t* base, int64_t ld, int first, int rows, int end) {
    const int n = end - first < 0 ? 0 : (end - first < rows ? end - first : rows);
    set(d, base + (int64_t)(n > 0 ? first : 0) * ld + (int64_t)k_first * BK, (uint32_t)n * (uint32_t)(ld * 2));
  };
  int w_left = 0;                                     // DH: rows of W from the wave's first one on
  auto w_bytes = [&]() {
    const int b = (w_left < 16 ? w_left : 16) * (int)res_ld2 - res0 * 2;
    return (uint32_t)(b > 0 ? b : 0);
  };
  if (RES_KMAJOR) {
    const int first = k_first * BK + wave * 16;
    w_left = p.V - first;
    set(dres, res_ptr + (int64_t)first * res_ld + res0, w_bytes());
  } else {
    rows_of(dres, res_ptr, res_ld, res0 + wave * 64, 64, MODE == MODE_FWD ? p.M : p.N);
  }
  if (RING_KMAJOR) set(dring, ring_ptr + ((int64_t)k_first * BK + wave * 16) * ring_ld + ring0, 16 * ring_ld2);
  else rows_of(dring, ring_ptr, ring_ld, ring0 + wave * (NJ * 8), NJ * 8, ring_end);
  // Five wait states between a vector instruction that writes a scalar register (readfirstlane in `set`) and a load that reads it:
  // the compiler keeps them for its own loads only.  (In the loop the descriptors are moved by scalar instructions.)
  asm volatile("s_nop 4" : "+s"(dres), "+s"(dring));
  uint32_t slot = lds_wave;                           // of the panel being loaded
  int loading = 0;
  auto load = [&](int l) {
    if (l < 8) load_lds16(vres[kind(l)], from[l], dres, slot, to[l]); else load_lds16(vring[kind(l)], from[l], dring, slot, to[l]);
  };
  // to the next panel: the loads' slot and operands, in four pieces
  auto next_load_panel = [&](int piece) {
    if (piece == 0) { ++loading; slot = slot == lds_wave + (kSlots - 1) * kSlot ? lds_wave : slot + kSlot; }
    if (piece == 1) {
      if (RES_KMAJOR) { move(dres, (int64_t)res_ld2 * BK); w_left -= BK; }
      else move(dres, BK * 2 + (MODE == MODE_FWD && loading == p.a_tail_panel ? p.a_tail_delta : 0));
    }
    if (piece == 2) move(dring, RING_KMAJOR ? (int64_t)ring_ld2 * BK : BK * 2);
    if (piece == 3) {
      if (RES_KMAJOR) dres[2] = w_bytes();
      if (loading >= nk) { dres[2] = 0; dring[2] = 0; }   // behind the end nothing is fetched
    }
  };

  // ---- fragment reads
  int res_off[2], ring_off[2];                        // row-major: by K step; K-major: [0], and for ring blocks from 8 on [1]
  const int kr = 8 * fq + (frow >> 2);
  const int tr_col = ((frow & 2) << 3) + ((frow & 1) << 3);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int chunk = (ks << 2) | fq;
    if (RES_KMAJOR) res_off[ks] = (kr >> 4) * kWave + (kr & 15) * 512 + (kswz(kr) << 5) + tr_col + ws * 256;
    else if (MODE == MODE_FWD) res_off[ks] = ws * 2 * kWave + (8 * (frow >> 2) + (frow & 3)) * 128 + ((chunk ^ (((frow >> 1) & 1) | ((frow >> 2) << 1))) << 4);
    else res_off[ks] = ws * 2 * kWave + frow * 128 + ((chunk ^ ((frow >> 1) & 7)) << 4);
    if (RING_KMAJOR) ring_off[ks] = (kr >> 4) * kWave + 8192 + (kr & 15) * (NJ * 64) + tr_col + (ks == 0 ? wr * 256 + (kswz(kr) << 5) : 512 + ((kswz(kr) ^ (wr * 4)) << 5));
    else ring_off[ks] = wr * 2 * kWave + 8192 + frow * 128 + ((chunk ^ ((frow >> 1) & 7)) << 4);
  }
  auto read_tr = [&](int off, int four_rows) -> bf16x8 {
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4i16* lds_v4i16;
    unsigned char* q = smem + off;
    const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)q);
    const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(q + four_rows));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto read_res = [&](int i, int ks) -> bf16x8 {
    if (RES_KMAJOR) return read_tr((res_off[0] ^ (i << 5)) + ks * 2 * kWave, 2048);
    const int at = (i >> 2) * kWave + (MODE == MODE_FWD ? ((i >> 1) & 1) * 4096 + (i & 1) * 512 : (i & 3) * 2048);
    return *reinterpret_cast<const bf16x8*>(smem + res_off[ks] + at);
  };
  auto read_ring = [&](int j, int ks) -> bf16x8 {
    if (RING_KMAJOR) return read_tr((j < 8 ? ring_off[0] ^ (j << 5) : ring_off[1] ^ ((j - 8) << 5)) + ks * 2 * kWave, NJ * 256);
    return *reinterpret_cast<const bf16x8*>(smem + ring_off[ks] + j / ND * kWave + j % ND * 2048);
  };
  int read_slot = 0;                                  // the reads' slot: the ring's, and behind it the resident side's
  auto slot_step = [&]() { return read_slot == kSlots - 1 ? -(kSlots - 1) * kSlot : kSlot; };
  auto next_ring_panel = [&]() { ring_off[0] += slot_step(); ring_off[1] += slot_step(); };
  auto next_res_panel = [&]() {
    res_off[0] += slot_step();
    if (!RES_KMAJOR) res_off[1] += slot_step();
    read_slot = read_slot == kSlots - 1 ? 0 : read_slot + 1;
  };

  // ---- K loop
  f32x4 acc[NJ][8];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][i][e] = 0.f;
  bf16x8 res[8][2], ring[2][2][2];
#pragma unroll
  for (int s = 0; s < kSlots - 1; ++s) {
#pragma unroll
    for (int l = 0; l < kLoads; ++l) load(l);
#pragma unroll
    for (int q = 0; q < 4; ++q) next_load_panel(q);
  }
#pragma unroll
  for (int l = 0; l < kEarlyLoads; ++l) load(l);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm((kSlots - 2) * kLoads + kEarlyLoads));
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 20; ++q) {                      // (in the order of the loop, which is what its waits go by)
    if (q < 4) ring[0][q >> 1][q & 1] = read_ring(q >> 1, q & 1); else res[(q - 4) >> 1][q & 1] = read_res((q - 4) >> 1, q & 1);
    __builtin_amdgcn_sched_barrier(0);
  }
  int kt = 0;
  do {                                                // (at least one panel, as every caller has)
#pragma unroll
    for (int D = 0; D < ND; ++D) {
#pragma unroll
      for (int m = 0; m < 32; ++m) {
        const int i = m >> 2, jj = (m >> 1) & 1, ks = m & 1, j = 2 * D + jj, at = 32 * D + m;
        const bf16x8 &a = MODE == MODE_DH ? ring[D & 1][jj][ks] : res[i][ks], &b = MODE == MODE_DH ? res[i][ks] : ring[D & 1][jj][ks];
        if (j < 8) mfma16(acc[j][i], a, b); else mfma16_v(acc[j][i], a, b);
        const int since = at >= kBarrier ? at - kBarrier : at + kPanel - kBarrier;    // products since the last barrier
        if (since == 0) {
          __builtin_amdgcn_s_waitcnt(waitcnt_vm((kSlots - 2) * kLoads));
          __syncthreads();
        }
        if (D < ND - 1) {
          if (m < 4) ring[(D + 1) & 1][m >> 1][m & 1] = read_ring(2 * (D + 1) + (m >> 1), m & 1);
        } else {
          if (m >= 4 && m < 8) ring[0][(m - 4) >> 1][m & 1] = read_ring((m - 4) >> 1, m & 1);
          // a resident block is read again behind its last product
          if (m >= 8 && m < 12) res[(m - 8) >> 1][m & 1] = read_res((m - 8) >> 1, m & 1);
          if (m >= 12 && m < 30 && (m & 2) == 0) res[(m - 4) >> 2][m & 1] = read_res((m - 4) >> 2, m & 1);
          if (m == 31) { res[7][0] = read_res(7, 0); res[7][1] = read_res(7, 1); }
        }
        if (since >= kFirst && (since - kFirst) % kGap == 0 && (since - kFirst) / kGap < kLoads) load((since - kFirst) / kGap);
        if (since >= kPanel - 14 && since < kPanel - 2 && (since - kPanel + 14) % 3 == 0) next_load_panel((since - kPanel + 14) / 3);
        if (at == kPanel - 64 + 6) next_ring_panel();   // (behind the panel's last ring read)
        if (since == kPanel - 1) next_res_panel();
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  } while (++kt < nk);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));          // no direct load may outlive the wave
  // (the wait states between the last products and the first ordinary read of them)
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int j = 8; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(acc[j][i]));
  auto read_acc = [&](int j, int i, int e) { if (j < 8) return acc_now(acc[j][i][e]); return acc[j][i][e]; };

  if (MODE == MODE_FWD) {
    const Params& q = args_now();
    const int n0 = ring0 + wr * (NJ * 16), f = lane_now() & 15;
    float zt[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) { const int n = n0 + j * 16 + f; zt[j] = q.zt[n < ring_end ? n : ring_end - 1]; }
    // (here: else the compiler, which takes the tile bodies for ones that may follow each other, waits for these inside the loop of another
    // one, and with that for the panels on their way: 300 rows, V = 151936, d = 1536 195 us, now 182)
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    forward_epilogue<NJ>(q, [&](int i, int j, int e) { return read_acc(j, i, e); }, [&](int j) { return zt[j]; }, res0 + ws * 128, n0, res_tile * 2 + ws, ring_end);
  }
  if (MODE == MODE_DH) dh_epilogue<NJ>(p, smem, read_acc, wave, ring0 + wr * (NJ * 16), wr * (NJ * 16), res0 + ws * 128, ws * 128, ring_end, tail_out);
  if (MODE == MODE_DW) dw_epilogue<NJ>(p, acc, wr, ring0, res0 + ws * 128, res0, ring_end, tail_out);
}

// ---------------------------------------------------------------------------------------------
// 256 x 256 tiles: where they end earlier than tiles of 384 (see Cut and launch_gemm_dw_bf16).  Waves 2 x 2, each
// 128 x 128; the fragments of a panel's B side stay in registers, in two sets, and those of A go through a ring of four pairs; two
// panels of LDS.  (tile_product with 8 ring blocks takes 1 - 3 % longer: its resident fragments are all read again
// within the last 28 products of a panel.  dH of 2000 rows, d = 4096, V = 151936 1750 us with it and 1703, V = 32000 380 and 371.)
//   group 0      : A fragments of row block 3 (this panel); the last loads of the next panel's slot
//   groups 1 - 4 : A fragments of row blocks 4 - 7
//   group 5      : wait for this thread's part of panel kt+1, barrier; next panel's A block 0, B blocks 0 - 2; the first
//                  loads of panel kt+2 into this panel's slot
//   group 6      : next A block 1, B blocks 3 - 5, loads
//   group 7      : next A block 2, B blocks 6 - 7, loads
// FWD: A = W, rows permuted within fragments, B = token rows.  DH: A = rows of the stash, B = W^T from the rows of W (K-major, through a
// descriptor that ends with row V - 1: beyond it zeros are fetched).  DW: A = stash^T from its rows (K-major), B = rows of Ht; the
// MFMA's operands are swapped.  Panels k_first .. k_first + nk - 1, an even number, at least two.
// ---------------------------------------------------------------------------------------------
constexpr int TILE_BYTES = RES * BK * 2;               // one panel of 256 rows
constexpr int STAGE_BYTES = 2 * TILE_BYTES, PIPE_BYTES = 2 * STAGE_BYTES;
static_assert(PIPE_BYTES + RES * 4 <= tile_lds<kWide>(), "two panels and the tile's target logits");
constexpr int kLoadsInGroup[8] = {4, 0, 0, 0, 0, 4, 4, 4};
constexpr int load_index_base(int g) {      // loads issued before group g, in the order 5, 6, 7, 0, 1, ...
  int n = 0;
  for (int h = 5; h != g; h = (h + 1) & 7) n += kLoadsInGroup[h];
  return n;
}
constexpr int kLoadsCarriedOver = kLoadsInGroup[0] + kLoadsInGroup[1] + kLoadsInGroup[2] + kLoadsInGroup[3] + kLoadsInGroup[4];
static_assert(kLoadsCarriedOver + kLoadsInGroup[5] + kLoadsInGroup[6] + kLoadsInGroup[7] == 16, "a slot takes 16 loads per wave");

// A rows m0 .. M - 1 (at most 256), B rows n0 .. N - 1.  Workgroups that share a panel walk its row blocks in a different cyclic order
// (rot_a, rot_b), so that they do not all ask the L2 for the same lines at the same moment.
template <int MODE>
__device__ __forceinline__ void square_tile(const Params& p, unsigned char* smem, int m0, int M, int n0, int N, int rot_a, int rot_b, int part,
                                            int k_first, int nk, float* tail_out) {
  constexpr bool A_KMAJOR = MODE == MODE_DW, B_KMAJOR = MODE == MODE_DH;
  // (wave-uniform all of them; some come out of integer divisions, which run on the vector unit)
  m0 = __builtin_amdgcn_readfirstlane(m0); n0 = __builtin_amdgcn_readfirstlane(n0);
  k_first = __builtin_amdgcn_readfirstlane(k_first); nk = __builtin_amdgcn_readfirstlane(nk);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1, frow = lane & 15, fq = lane >> 4;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  // (opaque: else they are read again inside the loop, and the wait for that is one for every LDS read)
  int tail_panel = MODE == MODE_FWD ? p.a_tail_panel : 0;
  int64_t tail_delta = MODE == MODE_FWD ? p.a_tail_delta : 0;
  if (MODE == MODE_FWD) asm volatile("" : "+s"(tail_panel), "+s"(tail_delta));
  const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(lds_base + wave * 8192);
  const uint16_t* a_ptr[8];
  const uint16_t* b_ptr[8];
  uint32_t b_voff[8];                                 // DH: byte offset of the lane's chunk from the wave's 16 rows of W
  uint32_t lds_a[8], lds_b[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int ia = (i + rot_a) & 7, ib = (i + rot_b) & 7;
    lds_a[i] = __builtin_amdgcn_readfirstlane(ia * 1024);
    lds_b[i] = __builtin_amdgcn_readfirstlane(ib * 1024);
    const int r = (wave * 8 + ia) * 8 + (lane >> 3), rB = (wave * 8 + ib) * 8 + (lane >> 3);
    if (A_KMAJOR) {
      const int k = 2 * (wave * 8 + ia) + (lane >> 5);
      const int col = m0 + (((lane & 31) ^ (kswz(k) << 1)) << 3);     // (columns from V on: products that are not stored)
      a_ptr[i] = p.A + ((int64_t)k_first * BK + k) * p.lda + (col < p.V ? col : m0);
    } else {
      const int ra = m0 + r < M ? m0 + r : M - 1;
      const int chunk = MODE == MODE_FWD ? (lane & 7) ^ (((r >> 1) & 1) | (((r >> 3) & 3) << 1)) : (lane & 7) ^ ((r >> 1) & 7);
      a_ptr[i] = p.A + (int64_t)ra * p.lda + chunk * 8 + (int64_t)k_first * BK;
    }
    if (B_KMAJOR) {
      const int k = 2 * ib + (lane >> 5);
      b_voff[i] = (uint32_t)k * (uint32_t)(p.ldb * 2) + (((lane & 31) ^ (kswz(wave * 16 + k) << 1)) << 4);
    } else {
      const int rb = n0 + rB < N ? n0 + rB : N - 1;
      b_ptr[i] = p.B + (int64_t)rb * p.ldb + ((lane & 7) ^ ((rB >> 1) & 7)) * 8 + (int64_t)k_first * BK;
    }
  }
  const int64_t a_kstep = A_KMAJOR ? p.lda * (BK * 2) : BK * 2, w_kstep = p.ldb * (BK * 2);    // bytes per panel
  auto load_at = [](const uint16_t* base, int64_t byte_off, uint32_t lds) {
    uint64_t addr;
    asm volatile("s_mov_b32 m0, %3\n\tv_lshl_add_u64 %0, %1, 0, %2\n\tglobal_load_lds_dwordx4 %0, off"
                 : "=&v"(addr) : "v"(base), "s"(byte_off), "s"(lds) : "memory");
  };
  // DH: the wave's 16 rows of W in the panel being loaded
  uint64_t w_addr = 0;
  int w_left = 0;
  u32x4 w_desc = {0, 0, 0, 0x00020000u};
  auto w_set = [&]() {
    const int bytes = (w_left < 16 ? w_left : 16) * (int)(p.ldb * 2) - n0 * 2;    // (below 2^25: ldb is at most 2^20)
    w_desc[0] = (uint32_t)w_addr; w_desc[1] = (uint32_t)(w_addr >> 32);
    w_desc[2] = (uint32_t)(bytes > 0 ? bytes : 0);
  };
  auto w_advance = [&]() { w_addr += (uint64_t)w_kstep; w_left -= BK; w_set(); };
  if (B_KMAJOR) {
    const int first = k_first * BK + wave * 16;
    w_addr = (uint64_t)(p.B + (int64_t)first * p.ldb + n0);     // (uniform: the wave's number and the tile's are)
    w_left = p.V - first;
    w_set();
    asm volatile("s_nop 4" : "+s"(w_desc));           // (wait states in front of the first load, as in tile_product)
  }
  auto load_w = [](uint32_t voff, const u32x4& desc, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" :: "v"(voff), "s"(desc), "s"(lds) : "memory");
  };
  auto issue_range = [&](int kt, int slot, int j0, int j1) {
    const int64_t off = (int64_t)kt * (BK * 2), a_off = kt * a_kstep + (MODE == MODE_FWD && kt >= tail_panel ? tail_delta : 0);
#pragma unroll
    for (int j = j0; j < j1; ++j) {
      const uint32_t st = slot * STAGE_BYTES + wave_lds;
      if (B_KMAJOR && (j & 1)) load_w(b_voff[j >> 1], w_desc, st + TILE_BYTES + lds_b[j >> 1]);
      else if (j & 1) load_at(b_ptr[j >> 1], off, st + TILE_BYTES + lds_b[j >> 1]);
      else load_at(a_ptr[j >> 1], a_off, st + lds_a[j >> 1]);
    }
  };
  int a_off[2], b_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int chunk = (ks << 2) | fq;
    if (MODE == MODE_FWD) a_off[ks] = (wm * 128 + 8 * (frow >> 2) + (frow & 3)) * 128 + ((chunk ^ (((frow >> 1) & 1) | ((frow >> 2) << 1))) << 4);
    else a_off[ks] = (wm * 128 + frow) * 128 + ((chunk ^ ((frow >> 1) & 7)) << 4);
    b_off[ks] = TILE_BYTES + (wn * 128 + frow) * 128 + ((chunk ^ ((frow >> 1) & 7)) << 4);
  }
  // K-major panel: the transposing LDS read hands lane (g = lane / 16, s = lane % 16) the four
  // k values kb .. kb+3 of column m = mb + s when lane s points at row kb + s/4, columns
  // mb + 4*(s%4) .. +3.  Two of them (kb = 8g and 8g + 4 within the K step) make the lane's
  // 8-element fragment.
  const int kr = 8 * fq + (frow >> 2);
  const int tr = kr * 512 + (kswz(kr) << 5) + ((frow & 2) << 3) + ((frow & 1) << 3);
  const int a_tr = tr + wm * 256, b_tr = tr + wn * 256;
  auto read_tr = [&](int off) -> bf16x8 {
    typedef short v4i16 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) v4i16* lds_v4i16;
    unsigned char* q = smem + off;
    const v4i16 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)q);
    const v4i16 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16)(q + 2048));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto read_a = [&](int st, int ks, int i) -> bf16x8 {
    if (A_KMAJOR) return read_tr(st + (a_tr ^ (i << 5)) + ks * 16384);
    return *reinterpret_cast<const bf16x8*>(smem + st + a_off[ks] + (MODE == MODE_FWD ? (i >> 1) * 4096 + (i & 1) * 512 : i * 2048));
  };
  auto read_b = [&](int st, int ks, int j) -> bf16x8 {
    if (B_KMAJOR) return read_tr(st + TILE_BYTES + (b_tr ^ (j << 5)) + ks * 16384);
    return *reinterpret_cast<const bf16x8*>(smem + st + b_off[ks] + j * 2048);
  };
  f32x4 acc[8][8];
  bf16x8 fbx[2][2][8];   // [set][K step][16-column block]
  bf16x8 fax[4][2];      // [ring slot][K step]
  auto side = [&](int g, int m, int set, int st_cur, int st_nxt, int kt_nxt, int slot_nxt, int kt_load, int slot_cur) {
    int nr = 2;
    if (g == 0) {
      if (m < 2) fax[3][m] = read_a(st_cur, m, 3);
    } else if (g <= 4) {
      if (m < 2) fax[(g - 1) & 3][m] = read_a(st_cur, m, g + 3);
      if (B_KMAJOR && g == 4 && m == 6) w_advance();
    } else {
      const int q = g - 5, nb = q == 2 ? 2 : 3;       // B blocks read in this group
      if (g == 5 && m == 0) {
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
        __syncthreads();
      }
      if (m >= 1 && m < 3) fax[q][m - 1] = read_a(st_nxt, m - 1, q);
      if (m >= 3 && m < 3 + 2 * nb) { const int j = 3 * q + (m - 3) / 2, ks = (m - 3) & 1; fbx[set ^ 1][ks][j] = read_b(st_nxt, ks, j); }
      nr = 3 + 2 * nb;
    }
    const int nl = kLoadsInGroup[g];
    if (nl > 0 && m >= nr) {
#pragma unroll
      for (int i = 0; i < nl; ++i)
        if (m == nr + i * (16 - nr) / nl) {
          const int l = load_index_base(g) + i;
          if (g >= 5) issue_range(kt_load, slot_cur, l, l + 1); else issue_range(kt_nxt, slot_nxt, l, l + 1);
        }
    }
  };
  auto panel = [&](int set, int st_cur, int st_nxt, int kt_nxt, int slot_nxt, int kt_load, int slot_cur) {
#pragma unroll
    for (int g = 0; g < 8; ++g)
#pragma unroll
      for (int m = 0; m < 16; ++m) {
        const bf16x8 &a = fax[g & 3][m & 1], &b = fbx[set][m & 1][m >> 1];
        if (MODE == MODE_DW) mfma16(acc[g][m >> 1], b, a); else mfma16(acc[g][m >> 1], a, b);
        side(g, m, set, st_cur, st_nxt, kt_nxt, slot_nxt, kt_load, slot_cur);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  auto last_k = [&](int k) { return k < nk ? k : nk - 1; };
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
  issue_range(0, 0, 0, 16);
  if (B_KMAJOR) w_advance();
  if (MODE == MODE_FWD) {
    const int n = n0 + wave * 64 + lane;              // the tile's target logits, published with its first panel
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off"
                 :: "v"(p.zt + (n < N ? n : N - 1)), "s"(__builtin_amdgcn_readfirstlane(lds_base + PIPE_BYTES + wave * 256)) : "memory");
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  __syncthreads();
  issue_range(last_k(1), 1, 0, 16 - kLoadsCarriedOver);   // the rest comes with the first groups of the first panel
#pragma unroll
  for (int q = 0; q < 3; ++q) {                       // (in the order of the loop, which is what its waits go by)
#pragma unroll
    for (int m = 0; m < (q == 2 ? 6 : 8); ++m) {
      const int j = 3 * q + (m - 2) / 2;
      if (m < 2) fax[q][m] = read_a(0, m, q); else fbx[0][m & 1][j] = read_b(0, m & 1, j);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  int kt = 0;
  do {
    panel(0, 0, STAGE_BYTES, last_k(kt + 1), 1, last_k(kt + 2), 0);
    panel(1, STAGE_BYTES, 0, last_k(kt + 2), 0, last_k(kt + 3), 1);
    kt += 2;
  } while (kt < nk);
  __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));          // no direct load may outlive the wave
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
  auto read_acc = [&](int i, int j, int e) { return acc_now(acc[i][j][e]); };
  if (MODE == MODE_FWD) {
    const unsigned char* const zt_lds = smem + PIPE_BYTES + ((wn * 128 + (lane_now() & 15)) << 2);
    forward_epilogue<8>(p, read_acc, [&](int j) { return *reinterpret_cast<const float*>(zt_lds + j * 64); }, m0 + wm * 128, n0 + wn * 128, part * 2 + wm, N);
  }
  if (MODE == MODE_DH) dh_epilogue<8>(p, smem, read_acc, wave, m0 + wm * 128, wm * 128, n0 + wn * 128, wn * 128, M, tail_out);
  if (MODE == MODE_DW) dw_epilogue<8>(p, acc, wm, m0, n0 + wn * 128, n0, M, tail_out);
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
  const Params& p = args_now();
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1, frow = lane & 15, fq = lane >> 4;
  const int m0 = tm * RES, M = p.M, nk = p.K / BK;
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
  // (opaque: else they are read again inside the loop, and the wait for that is one for every LDS read)
  int tail_panel = p.a_tail_panel;
  int64_t tail_delta = p.a_tail_delta;
  asm volatile("" : "+s"(tail_panel), "+s"(tail_delta));
  // load l of panel kt (behind the end: the last one again, into a slot nobody reads)
  auto load = [&](int l, int kt, uint32_t stage) {
    kt = kt < nk ? kt : nk - 1;
    const int64_t off = (int64_t)kt * (BK * 2) + (l < 8 && kt >= tail_panel ? tail_delta : 0);
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
  forward_epilogue<4>(p, [&](int i, int j, int e) { return acc_now(acc[i][j][e]); },
                      [&](int j) { return *reinterpret_cast<const float*>(zt_lds + j * 64); }, m0 + wm * 128, n0 + wn * 64, tm * 2 + wm, N);
}

// No panels at all: a slice of the contraction that the plan did not need, or dW without a scored row.
__device__ inline void zero_rows(float* at, int64_t ld, int rows, int cols) {
  for (int r = threadIdx.x >> 6; r < rows; r += NTHREADS / 64)
    for (int c = (threadIdx.x & 63) * 4; c < cols; c += 256) *reinterpret_cast<f32x4_any*>(at + (int64_t)r * ld + c) = f32x4{0.f, 0.f, 0.f, 0.f};
}

__host__ __device__ __forceinline__ int tiles_of(int n, int size) { return (n + size - 1) / size; }

// How n token rows (columns of forward tiles, rows of dH tiles) are cut into tiles of 384, 256 and 128.  The host says for every count of rows
// up to 16384, in steps of 128, which of three ways it is (Params::cuts): the scored rows are known on the device only, and a choice
// made there cost every tile of a short launch a microsecond and more.
struct Cut {
  int wide, narrow, half;
  __host__ __device__ __forceinline__ int count() const { return wide + narrow + half; }
  __host__ __device__ __forceinline__ int start(int t) const {
    return t < wide ? t * RING : t < wide + narrow ? wide * RING + (t - wide) * 256 : wide * RING + narrow * 256 + (t - wide - narrow) * 128;
  }
  __host__ __device__ __forceinline__ int blocks(int t) const { return t < wide ? kWide : t < wide + narrow ? 8 : 4; }   // of 16 rows per wave
};
// Tiles of 384 and what is left; two of 256 instead of one of 384 and one of 128, which waits for its panels more than it computes.
__host__ __device__ __forceinline__ Cut cut_wide(int n) {
  const int w = n / RING, r = n - w * RING;
  if (r == 0) return {w, 0, 0};
  if (r <= 128) return w ? Cut{w - 1, 2, 0} : Cut{0, 0, 1};
  return r <= 256 ? Cut{w, 1, 0} : Cut{w + 1, 0, 0};
}
__host__ __device__ __forceinline__ Cut cut_narrow(int n) {
  const int w = n / 256, r = n - w * 256;
  return r == 0 ? Cut{0, w, 0} : r <= 128 ? Cut{0, w, 1} : Cut{0, w + 1, 0};
}
constexpr int kCutStep = 128, kCutSteps = 128;
enum { CUT_WIDE = 0, CUT_NARROW = 1, CUT_SHORT = 2, CUT_EVEN = 3 };
// CUT_NARROW: of 256, and in the forward one of 128; CUT_SHORT: forward a last tile of 384 as one of 256 and one of 128, dH all of 128; CUT_EVEN: all of 256.
template <int MODE> __host__ __device__ __forceinline__ Cut cut_rows(int n, int kind) {
  if (kind == CUT_WIDE) return cut_wide(n);
  if (kind == CUT_EVEN) return Cut{0, tiles_of(n, 256), 0};
  if (MODE == MODE_FWD) return kind == CUT_NARROW ? cut_narrow(n) : Cut{tiles_of(n, RING) - 1, 1, 1};
  return Cut{0, 0, tiles_of(n, 128)};
}
__host__ __device__ __forceinline__ int cut_kind(const uint64_t (&cuts)[4], int n) {
  const int i = (n - 1) / kCutStep;                   // (all four words read and selected from: every tile 0.3 us later)
  return i < kCutSteps ? (int)(cuts[i >> 5] >> (2 * (i & 31))) & 3 : CUT_WIDE;
}
template <int MODE> __device__ __forceinline__ Cut cut_of(const Params& p, int n) { return cut_rows<MODE>(n, cut_kind(p.cuts, n)); }

__device__ __forceinline__ int dh_band(const Cut& cut) { return cut.wide > 0 ? 4 : 8; }

template <int MODE>
__global__ __launch_bounds__(NTHREADS) void gemm_nt_bf16(Params p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // valid rows of this chunk (device-side, no host sync)
  const int64_t nv64 = *p.n_scored - p.chunk_start;
  const int nvalid = __builtin_amdgcn_readfirstlane(nv64 < 0 ? 0 : (nv64 > p.chunk_rows ? p.chunk_rows : (int)nv64));
  if (nvalid == 0 && (MODE != MODE_DW || !p.overwrite)) return;
  int tm, tn;
  if constexpr (MODE == MODE_FWD) {
    const int Mt = tiles_of(p.M, RES);
    const Cut cut = cut_of<MODE>(p, nvalid);
    const int Nt = cut.count();
    if (!dealt_tile(8, blockIdx.x, Mt, Nt, tm, tn)) return;
    if (cut.half > 0 && Nt > 1) {
      // half tiles are dealt like the others, to every XCD its share: the columns of a band start at another one in every
      // band (with 8 columns, XCDs would else have all of them or none)
      tn += tm / 8 % Nt;
      tn = tn < Nt ? tn : tn - Nt;
    }
    const int n0 = cut.start(tn), blocks = cut.blocks(tn);
    // (the arguments as they are in the short one's: read again they are two scalar latencies a tile, 1 % at 8 panels)
    if (blocks == 4) half_column_tile(smem, tm, n0, nvalid);
    else if (__builtin_expect(blocks == 8, 1))
      square_tile<MODE>(p, smem, tm * RES, p.M, n0, nvalid < n0 + 256 ? nvalid : n0 + 256, 2 * tn & 7, tm & 7, tm, 0, p.K / BK, nullptr);
    else tile_product<MODE, kWide>(p, smem, tn, tm, n0, nvalid, 0, p.K / BK, nullptr);
  } else if constexpr (MODE == MODE_DH) {
    const int Nt = tiles_of(p.N, RES);
    const Cut cut = cut_of<MODE>(p, nvalid);
    const int Mt = cut.count(), panels = p.K / BK;
    int k_first = 0, nk = panels;
    float* tail_out = nullptr;
    const int item = split_tile(dh_band(cut), blockIdx.x, Mt, Nt, panels, p.max_items, DhSplit{}, tm, tn, k_first, nk);
    if (item < -1) return;
    if (item >= 0) {
      tail_out = p.tail_part + (int64_t)item * (RING * RES);
      if (nk <= 0) { zero_rows(tail_out, RES, RING, RES); return; }
    }
    const int m0 = cut.start(tm), blocks = cut.blocks(tm);
    if (blocks == 4) tile_product<MODE, 4>(p, smem, tm, tn, m0, nvalid < m0 + 128 ? nvalid : m0 + 128, k_first, nk, tail_out);
    else if (blocks == 8) square_tile<MODE>(p, smem, m0, nvalid < m0 + 256 ? nvalid : m0 + 256, tn * RES, p.N, 2 * tn & 7, tm & 7, 0, k_first, nk, tail_out);
    else tile_product<MODE, kWide>(p, smem, tm, tn, m0, nvalid, k_first, nk, tail_out);
  } else if (p.wide) {
    const int panels = dw_panels(nvalid, p.K), Mt = tiles_of(p.V, RING), Nt = tiles_of(p.d, RES);
    int k_first = 0, nk = panels;
    const int item = split_tile(4, blockIdx.x, Mt, Nt, panels, p.max_items, DwSplit{}, tm, tn, k_first, nk);
    if (item < -1 || (item >= 0 && nk <= 0)) return;  // (an empty slice: nothing to store, and nobody reads it)
    const int rows = p.V - tm * RING < RING ? p.V - tm * RING : RING, cols = p.d - tn * RES < RES ? p.d - tn * RES : RES;
    if (panels == 0) zero_rows(p.dW + (int64_t)tm * RING * p.d + tn * RES, p.d, rows, cols);
    else tile_product<MODE, kWide>(p, smem, tm, tn, tm * RING, p.V, k_first, nk, item >= 0 ? p.tail_part + (int64_t)item * (RING * RES) : nullptr);
  } else {
    // 256 x 256 tiles: the rows of tiles up to the tail's first one, and the tail's slices (see dw_tail_plan)
    const int panels = dw_panels(nvalid, p.K), Nt = tiles_of(p.d, RES);
    const int Mt = p.tail_split > 0 ? p.tail_m0 : tiles_of(p.V, RES);
    int k_first = 0, nk = panels;
    float* tail_out = nullptr;
    if (p.tail_split == 0 || (int)blockIdx.x < p.main_blocks) {
      if (!tile_coords(blockIdx.x, Mt, Nt, p.sup_m, p.sup_n, tm, tn)) return;
      if (panels == 0) {
        zero_rows(p.dW + (int64_t)tm * RES * p.d + tn * RES, p.d, p.V - tm * RES < RES ? p.V - tm * RES : RES, p.d - tn * RES < RES ? p.d - tn * RES : RES);
        return;
      }
    } else {
      // one XCD takes consecutive items (the host says how many: the XCDs that the whole tiles
      // leave idle earlier take more), i.e. mostly tiles of one slice: they walk the same K range
      // and share its operand panels in that L2
      const int e = blockIdx.x - p.main_blocks, tiles = p.tail_rows * Nt;
      const int item = p.tail_first[e % NXCD] + e / NXCD;
      if (item >= p.tail_first[e % NXCD + 1]) return;
      const int slice = item / tiles, t = item % tiles, per = slice_panels(panels, p.tail_split);
      if (slice >= slices_in_use(panels, p.tail_split)) return;   // empty: nothing to store, and nobody reads it
      tm = p.tail_m0 + t / Nt; tn = t % Nt;
      k_first = slice * per;
      nk = panels - k_first < per ? panels - k_first : per;
      tail_out = p.tail_part + (int64_t)item * (RES * RES);
      if (nk <= 0) { zero_rows(tail_out, RES, RES, RES); return; }
    }
    square_tile<MODE>(p, smem, tm * RES, p.V, tn * RES, p.N, tn * 8 / p.sup_n & 7, tm * 8 / p.sup_m & 7, 0, k_first, nk, tail_out);
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
  forward_epilogue<4>(p, [&](int i, int j, int e) { return acc_now(acc[i][j][e]); }, [&](int j) { return zt[j]; }, m0, wave * 64, tm, N);
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
  if (!dealt_tile(8, blockIdx.x, Mt, Nt, tm, tn)) return;
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
struct DwTailPlan { int m0, rows, split, first[NXCD + 1]; double end; };   // end: of the launch, in tile times
DwTailPlan dw_tail_plan(int Mt, int Nt, int sup_m, int sup_n) {
  constexpr double kItemOverhead = 0.02;         // prologue, partial-tile store, reduce: in tile times
  DwTailPlan best = {Mt / sup_m * sup_m, Mt % sup_m, 0, {}, 0};
  const int tiles = best.rows * Nt;
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
  best.end = unsplit;
  if (tiles == 0 || best.m0 == 0) return best;
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
      best_end = best.end = end; best.split = split; best.first[0] = 0;
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
  const int t = (int)(q / (RES * RES)), within = (int)(q % (RES * RES));
  if (t >= tiles) return;
  const int v = (tail_m0 + t / Nt) * RES + within / RES, n = (t % Nt) * RES + within % RES;
  if (v >= V || n >= d) return;
  float s = 0.f;
  const int slices = slices_in_use(dw_panels(nvalid, chunk_rows), split);
  for (int k = 0; k < slices; ++k) s += part[((int64_t)k * tiles + t) * (RES * RES) + within];
  float* out = dW + (int64_t)v * d + n;
  *out = overwrite ? s : *out + s;
}

// Adds the slices of the tiles that the dH launch cut (slice 0 first), applies the row scale and scatters the rows to their
// slots: 8 columns per thread.  Blocks beyond the tiles that the device finds cut return at once.
constexpr int kReduceBlocks = RING * RES / 2048;      // per tile
__device__ inline void add_slices(const float* part, int slices, int rest, int t, int within, f32x4& lo, f32x4& hi) {
  lo = hi = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int s = 0; s < slices; ++s) {
    const f32x4* q = reinterpret_cast<const f32x4*>(part + ((int64_t)s * rest + t) * (RING * RES) + within);
    lo += q[0];
    hi += q[1];
  }
}
__global__ __launch_bounds__(256) void dh_tail_reduce(Params p) {
  int64_t nv64 = *p.n_scored - p.chunk_start;
  const int M = nv64 < 0 ? 0 : (nv64 > p.chunk_rows ? p.chunk_rows : (int)nv64);
  const int Nt = tiles_of(p.N, RES);
  if (M == 0) return;
  const Cut cut = cut_of<MODE_DH>(p, M);
  const int Mt = cut.count();
  const int tiles = Mt * Nt, whole = tiles / kRound * kRound, rest = tiles - whole;
  const int t = blockIdx.x / kReduceBlocks;
  if (t >= rest) return;
  const int split = dh_split(rest, p.K / BK, p.max_items);
  if (split == 1) return;
  int tm, tn;
  tile_at(dh_band(cut), whole + t, Mt, Nt, tm, tn);
  const int within = (blockIdx.x % kReduceBlocks) * 2048 + threadIdx.x * 8;
  const int m = cut.start(tm) + within / RES, n = tn * RES + within % RES;
  if (within / RES >= 32 * cut.blocks(tm) || m >= M || n >= p.d) return;
  f32x4 lo, hi;
  add_slices(p.tail_part, split, rest, t, within, lo, hi);
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
// The same for the dW launch on 384 x 256 tiles.
__global__ __launch_bounds__(256) void dw_wide_reduce(Params p) {
  int64_t nv64 = *p.n_scored - p.chunk_start;
  const int nvalid = nv64 < 0 ? 0 : (nv64 > p.chunk_rows ? p.chunk_rows : (int)nv64);
  const int panels = dw_panels(nvalid, p.K);
  const int Mt = tiles_of(p.V, RING), Nt = tiles_of(p.d, RES), tiles = Mt * Nt, whole = tiles / kRound * kRound, rest = tiles - whole;
  const int split = dw_split(rest, panels, p.max_items);
  if (split == 1) return;
  int tm, tn;
  const int t = blockIdx.x / kReduceBlocks;
  tile_at(4, whole + t, Mt, Nt, tm, tn);
  const int within = (blockIdx.x % kReduceBlocks) * 2048 + threadIdx.x * 8;
  const int v = tm * RING + within / RES, n = tn * RES + within % RES;
  if (v >= p.V || n >= p.d) return;
  f32x4 lo, hi;
  add_slices(p.tail_part, slices_in_use(panels, split), rest, t, within, lo, hi);
  f32x4_any* const out = reinterpret_cast<f32x4_any*>(p.dW + (int64_t)v * p.d + n);
  if (!p.overwrite) { lo = out[0] + lo; hi = out[1] + hi; }
  out[0] = lo;
  out[1] = hi;
}

template <void (*KERNEL)(Params)> void launch(Params& p, int blocks, hipStream_t stream) {
  static LdsLimit lds_limit;
  lds_limit.ensure(reinterpret_cast<const void*>(KERNEL), tile_lds<kWide>());
  hipLaunchKernelGGL(KERNEL, dim3(blocks), dim3(NTHREADS), tile_lds<kWide>(), stream, p);
}
int tiles(int64_t n, int size) { return (int)((n + size - 1) / size); }

// When a forward launch of rows x c tiles over `panels` ends, in hundredths of a 256 x 256 tile's panel: whole rounds of the longest kind of tile, or where
// several kinds are earlier than that, the mean and a part of the longest.  A tile of 384 counts 1.34 and one of 128 0.53, and each 4 or 6 panels beyond its
// own; a single column of 384 streams its own rows of W from memory and waits for them.  Fitted to launches of 257 - 15900 rows over
// 14 heads, scoring and with the stash, each cut in all ways; what it picks takes 0.4 % longer than the best of them.  Scoring, us, tiles of 256 and 128, tiles
// of 384: V = 151936, d = 4096, 300 rows 422 and 413, 600 rows 648 and 622, 2500 rows 2249 and 2184; d = 1536, 300 rows 168 and 177, 900 rows 396 and 363; V = 50257,
// d = 712, 300 rows 47 and 36, 1280 rows 97 and 113; V = 32000, d = 4096, 300 rows 98 and 117, 600 rows 165 and 128; d = 1536, 2000 rows 154 and 166, 2100 rows 179 and
// 159; V = 8192, d = 4096, 1280 rows 78 and 109, 2500 rows 163 and 126.
// An even number of groups of four columns in a band puts the group with the shorter columns on the same XCDs in every band, and the others have whole rounds of
// the longest kind: no mean there (`apart`; 5633 - 5888 and 8705 - 8960 rows, with the mean, tiles of 384 and two columns of 256, and without it, tiles of 256:
// V = 20711, d = 2048 420 and 388, V = 45174 809 and 751, V = 30328, d = 1840 549 and 523, V = 5816, d = 1536 180 and 168, V = 74627, d = 496 468 and 461, V = 128256,
// d = 128 449 and 457). With eight columns the mean holds all the same (2814 rows, V = 151936, d = 744 595 with the mean, 648 without).
// (Worked out for every step of every launch, so what does not depend on the cut comes from outside: 120 steps 1.9 and 1.1 us of host time.)
struct ForwardTiles {
  int64_t wide, alone, narrow, half;
  explicit ForwardTiles(int panels) : wide(134 * (int64_t)panels + 600), alone(wide * 115 / 100), narrow(100 * (int64_t)panels + 400), half(53 * (int64_t)panels + 600) {}
};
int64_t forward_end(const Cut& c, int rows, const ForwardTiles& t) {
  const int count = c.count();
  const int64_t wide = count == 1 ? t.alone : t.wide, most = c.wide > 0 ? wide : c.narrow > 0 ? t.narrow : t.half;
  const uint64_t all = (uint64_t)count * rows;
  int64_t end = (int64_t)((all + kRound - 1) / kRound) * most;
  const bool apart = c.wide > 0 && c.half == 0 && count > 8 && count % 8 == 0;
  if (!apart && all > kRound && count != c.wide && count != c.narrow && count != c.half) {
    const int64_t work = (int64_t)((uint64_t)(c.wide * wide + c.narrow * t.narrow + c.half * t.half) * rows / kRound);
    const int64_t mixed = work + most * (c.wide > 0 ? 70 : 61) / 100;
    end = mixed < end ? mixed : end;
    end = end > most ? end : most;
  }
  return c.wide > 0 ? end + end / 50 : end;
}
// In a single round that fills most of the chip the last tile of a launch without tiles of 384 is a whole one: beside one of 128, which runs ahead of the one
// of 256 in the same rows of W, both read those from memory (300 rows, V = 32000, d = 2048 51 and 54 us, d = 4096 94 and 98, d = 8192 195 and 239; with 8 panels
// the same; fewer tiles V = 20000, d = 6144 120 and 114, V = 8000, d = 16384 305 and 283).
int forward_kind(int n, int rows, int panels, const ForwardTiles& t) {
  const Cut a = cut_wide(n), b = cut_narrow(n);
  const bool even = panels >= 16 && b.half > 0 && b.narrow > 0 && b.count() * rows <= kRound && b.count() * rows > kRound * 3 / 4;
  const int small = even ? CUT_EVEN : CUT_NARROW;
  if (a.wide == 0) return small;
  const int64_t ea = forward_end(a, rows, t), eb = forward_end(even ? cut_rows<MODE_FWD>(n, CUT_EVEN) : b, rows, t);
  const int64_t ec = a.count() == a.wide && a.wide > 1 ? forward_end(Cut{a.wide - 1, 1, 1}, rows, t) : ea;
  return eb <= ea && eb <= ec ? small : ec < ea ? CUT_SHORT : CUT_WIDE;
}

// When a dH launch of c x cols tiles over `panels` ends, in hundredths of a 256 x 256 tile's panel: whole rounds of 256 tiles, and the last round in as many
// slices as end earliest (a closed form of what dh_split searches for).  A tile of 384 counts 1.32 and one of 128 0.58, and a tile or slice 22
// panels beyond its own, which favours few long ones: fitted to launches of 64 - 5120 rows over 13 heads, each cut in all three ways.
int64_t dh_end(const Cut& c, int cols, int panels, int max_items) {
  constexpr int kWideTile = 132, kNarrowTile = 100, kHalfTile = 58, kExtra = 22;
  const int64_t all = (int64_t)c.count() * cols, whole = all / kRound;
  const int64_t mean = (c.wide * kWideTile + c.narrow * kNarrowTile + c.half * kHalfTile) / c.count();
  const int rest = (int)(all % kRound);
  const int64_t one = whole > 0 ? mean : c.wide ? kWideTile : c.narrow ? kNarrowTile : kHalfTile;
  int64_t last = 0;
  for (int rounds = 1; rest > 0 && rounds <= 3; ++rounds) {
    int s = rounds * kRound / rest;
    s = s < dh_most_split(panels) ? s : dh_most_split(panels);
    s = s * rest <= max_items ? s : max_items / rest;
    s = s > 1 ? s : 1;
    const int64_t e = tiles((int64_t)rest * s, kRound) * (int64_t)(slice_panels(panels, s) + kExtra) * one;
    last = rounds == 1 || e < last ? e : last;
  }
  return whole * (panels + kExtra) * mean + last;
}
// Tiles of 128 only up to one round of them.  us, launch and reduction, tiles of 384, 256 and 128: V = 8192, d = 512, 300 rows 41, 35 and 24, 4000 rows 59, 53
// and 46; V = 32000, d = 1536, 300 rows 61, 58 and 47, 900 rows 96, 92 and 90, 4000 rows 314, 344 and 365; d = 4096, 1500 rows 284, 322 and 389,
// 2000 rows 417, 371 and 417; V = 151936, 300 rows 352, 463 and 429, 2000 rows 1762, 1703 and 2007, 3000 rows 2384, 2670 and 3062.
int dh_kind(int n, int cols, int panels, int max_items) {
  const Cut w = cut_rows<MODE_DH>(n, CUT_WIDE), q = cut_rows<MODE_DH>(n, CUT_EVEN), h = cut_rows<MODE_DH>(n, CUT_SHORT);
  int64_t best = dh_end(w, cols, panels, max_items);
  int kind = CUT_WIDE;
  auto take = [&](const Cut& c, int k) { const int64_t e = dh_end(c, cols, panels, max_items); if (e < best) { best = e; kind = k; } };
  take(q, CUT_EVEN);
  if (h.half * cols <= kRound) take(h, CUT_SHORT);
  return kind;
}

// What the host settles for a launch: how every count of valid rows up to chunk_rows is cut (all counts of a step alike), and as many
// workgroups as any of them needs.
struct CutPlan { uint64_t cuts[4]; int blocks, most; };
template <class Kind> CutPlan plan_cuts(int rows, Kind kind) {
  CutPlan plan = {};
  for (int i = 0; i < kCutSteps && i * kCutStep < rows; ++i) plan.cuts[i >> 5] |= (uint64_t)kind((i + 1) * kCutStep) << (2 * (i & 31));
  return plan;
}
// The plan of the launch before, per thread: a call's passes and the parts of a pass are alike (1000000 slots, 100 scored, V = 1000, d = 64: 64 forward
// launches, 358 us a call without it and 349 with it).
struct LastPlan {
  int64_t key[4] = {-1, -1, -1, -1};
  CutPlan plan;
  template <class Make> const CutPlan& get(int64_t a, int64_t b, int64_t c, int64_t e, Make make) {
    if (key[0] != a || key[1] != b || key[2] != c || key[3] != e) { plan = make(); key[0] = a; key[1] = b; key[2] = c; key[3] = e; }
    return plan;
  }
};
CutPlan plan_forward(int chunk_rows, int V, int d) {
  const int Mt = tiles(V, RES), panels = (int)(round_up(d, 2 * BK) / BK);
  const ForwardTiles t(panels);
  CutPlan plan = plan_cuts(chunk_rows, [&](int n) { return forward_kind(n, Mt, panels, t); });
  plan.blocks = (int)round_up((int64_t)Mt * tiles(chunk_rows, 256), NXCD);
  return plan;
}
CutPlan plan_dh(int chunk_rows, int V, int d, int max_items) {
  const int Nt = tiles(d, RES), panels = (int)(round_up(V, 2 * BK) / BK);
  int most = cut_wide(chunk_rows).count() * Nt;       // tiles, whatever the count of scored rows
  CutPlan plan = plan_cuts(chunk_rows, [&](int n) {
    const int kind = dh_kind(n, Nt, panels, max_items), t = cut_rows<MODE_DH>(n, kind).count() * Nt;
    most = t > most ? t : most;
    return kind;
  });
  plan.most = most;
  plan.blocks = most / kRound * kRound + (int)round_up(dh_most_items(most, panels, max_items), NXCD);
  return plan;
}
// dW, passes above kFewDwRows: 384 x 256 tiles, or 256 x 256 ones where those end earlier (short contractions over few rounds of tiles, whose last round the
// cut does not pay for): 1.43 of the other tile's time, and about 8 panels' time per tile for its epilogue in either.
// Launch, us, 256 x 256 and 384 x 256: V = 151936, 65536 rows, d = 4096 53800 and 50960, 47360 rows, d = 3584 34074 and 30363, 5120 rows,
// d = 1536 1797 and 1675; V = 128256, 2000 rows, d = 1024 457 and 438.
struct DwPlan { bool wide; int tiles, rest, most_split, blocks; SuperTile super; DwTailPlan tail; };
DwPlan plan_dw(int chunk_rows, int expected_rows, int V, int d, int max_items) {
  const int Nt = tiles(d, RES), expected = tiles(expected_rows, BK), most_panels = chunk_rows / BK;
  DwPlan plan = {};
  plan.super = pick_super_tile(Nt);
  plan.tail = dw_tail_plan(tiles(V, RES), Nt, plan.super.m, plan.super.n);
  plan.tiles = tiles(V, RING) * Nt;
  plan.rest = plan.tiles % kRound;
  plan.most_split = 1;
  const int rest = plan.rest, split = rest > 0 ? dw_split(rest, expected, max_items) : 1;
  const double last = rest == 0 ? 0 : split == 1 ? expected + 6 : tiles(rest * split, kRound) * ((expected + split - 1) / split + 6) + 12;
  plan.wide = 1.43 * (plan.tiles / kRound * (expected + 6) + last) <= plan.tail.end * (expected + 8);
  if (plan.wide) {
    plan.blocks = plan.tiles;
    if (rest > 0 && most_panels >= 16) {              // (as many slices as any count of scored rows can make)
      plan.most_split = most_panels / 8 < 64 ? most_panels / 8 : 64;
      const int items = rest * plan.most_split < max_items ? rest * plan.most_split : max_items;
      plan.blocks = plan.tiles - rest + (items > rest ? items : rest);
    }
    plan.blocks = (int)round_up(plan.blocks, NXCD);
    return plan;
  }
  plan.blocks = num_blocks(plan.tail.split > 0 ? plan.tail.m0 : tiles(V, RES), Nt, plan.super.m, plan.super.n);
  return plan;
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
    const int Mt = 2 * tiles(p.M, RES);
    hipLaunchKernelGGL(forward_few_bf16, dim3(Mt), dim3(NTHREADS), F_LDS, stream, p);
    return;
  }
  thread_local LastPlan last;
  const CutPlan& plan = last.get(chunk_rows, V, d, 0, [&] { return plan_forward(chunk_rows, V, d); });
  std::memcpy(p.cuts, plan.cuts, sizeof p.cuts);
  launch<gemm_nt_bf16<MODE_FWD>>(p, plan.blocks, stream);
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
  thread_local LastPlan last;
  const CutPlan& plan = last.get(chunk_rows, V, d, tail_items, [&] { return plan_dh(chunk_rows, V, d, tail_items); });
  std::memcpy(p.cuts, plan.cuts, sizeof p.cuts);
  launch<gemm_nt_bf16<MODE_DH>>(p, plan.blocks, stream);
  if (dh_most_split(p.K / BK) > 1)
    hipLaunchKernelGGL(dh_tail_reduce, dim3((plan.most < kRound ? plan.most : kRound - 1) * kReduceBlocks), dim3(256), 0, stream, p);
}

size_t gemm_tail_tile_bytes() { return (size_t)RING * RES * sizeof(float); }
// One partial tile per compute unit for the dW launch; the dH launch's last round of up to 255 tiles can use up to four; a
// quarter of the size of the head, which has the longer tiles the larger it is, bounds the extra ones.
int gemm_tail_items(size_t head_bytes) {
  const size_t extra = head_bytes / 4 / ((size_t)RES * RES * sizeof(float));
  return kDwTailMaxItems + (int)(extra < 768 ? extra : 768);
}
// (as many of 256 x 256: what a workspace had before the tiles grew; their last round is then cut into fewer slices)
size_t gemm_tail_bytes_least(size_t head_bytes) { return (size_t)gemm_tail_items(head_bytes) * RES * RES * sizeof(float); }
bool dw_rows_in_blocks(int rows) { return rows <= kFewDwRows; }

void launch_gemm_dw_bf16(const void* E, int64_t lde, const void* Ht, int64_t ldht,
                         const int64_t* n_scored, int64_t chunk_start, int chunk_rows,
                         int V, int d, float* dW, int overwrite, float* tail_part, int tail_items, int rows, bool in_blocks,
                         hipStream_t stream) {
  Params p = {};
  p.A = static_cast<const uint16_t*>(E); p.lda = lde;
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
  p.max_items = tail_items;
  const DwPlan plan = plan_dw(chunk_rows, rows, V, d, tail_items);
  p.wide = plan.wide;
  if (p.wide) {
    launch<gemm_nt_bf16<MODE_DW>>(p, plan.blocks, stream);
    if (plan.most_split > 1) hipLaunchKernelGGL(dw_wide_reduce, dim3(plan.rest * kReduceBlocks), dim3(256), 0, stream, p);
    return;
  }
  const DwTailPlan& tail = plan.tail;
  const int Nt = tiles(d, RES);
  p.sup_m = plan.super.m; p.sup_n = plan.super.n;
  p.main_blocks = plan.blocks;
  int blocks = p.main_blocks;
  if (tail.split > 0) {
    p.tail_m0 = tail.m0; p.tail_rows = tail.rows; p.tail_split = tail.split;
    int most = 0;
    for (int x = 0; x < NXCD; ++x) {
      p.tail_first[x] = tail.first[x];
      most = tail.first[x + 1] - tail.first[x] > most ? tail.first[x + 1] - tail.first[x] : most;
    }
    p.tail_first[NXCD] = tail.first[NXCD];
    blocks += most * NXCD;
  }
  launch<gemm_nt_bf16<MODE_DW>>(p, blocks, stream);
  if (tail.split > 0) {
    const int n = tail.rows * Nt;
    hipLaunchKernelGGL(dw_tail_reduce, dim3(n * (RES * RES / 256)), dim3(256), 0, stream, tail_part, n, tail.split, Nt, tail.m0, V, d, dW,
                       overwrite, n_scored, chunk_start, chunk_rows);
  }
}

}  // namespace mrl

extern "C" int mrl_diag_dh_split(int32_t tail_tiles, int32_t panels, int32_t max_items) {
  using namespace mrl;
  if (tail_tiles <= 0 || tail_tiles >= kRound || panels <= 0 || max_items < tail_tiles) return MRL_ERR_SHAPE;
  return dh_split(tail_tiles, panels, max_items);
}

extern "C" int mrl_diag_dw_few_rows(void) { return mrl::kFewDwRows; }

extern "C" int mrl_diag_gemm_cut(int32_t launch, int32_t rows, int32_t expected, int32_t chunk_rows, int32_t V, int32_t d, int32_t tail_items,
                                 int32_t* out9) {
  using namespace mrl;
  if (out9 == nullptr) return MRL_ERR_NULL;
  if (V <= 0 || d <= 0 || d % 8 != 0 || chunk_rows <= 0 || chunk_rows % kTile != 0 || rows <= 0 || rows > chunk_rows || expected <= 0 ||
      tail_items < 0 || (launch != MRL_PROF_GEMM_FWD && launch != MRL_PROF_GEMM_DH && launch != MRL_PROF_GEMM_DW))
    return MRL_ERR_SHAPE;
  for (int i = 0; i < 9; ++i) out9[i] = 0;
  const int Nt = tiles(d, RES);
  const int items = tail_items > 0 ? tail_items : gemm_tail_items((size_t)round_up(d, 128) * (round_up(V, kTile) + 64) * 2);
  out9[7] = items;
  auto put = [&](int wide, int narrow, int half, int all, int split, int blocks) {
    out9[0] = wide; out9[1] = narrow; out9[2] = half; out9[3] = all;
    out9[4] = all % kRound; out9[5] = split; out9[6] = blocks;
  };
  if (launch == MRL_PROF_GEMM_DW) {
    if (dw_rows_in_blocks(expected)) return MRL_OK;
    const DwPlan plan = plan_dw(chunk_rows, expected, V, d, items);
    const int panels = dw_panels(rows, chunk_rows);
    if (plan.wide) put(tiles(V, RING), 0, 0, plan.tiles, plan.rest > 0 ? dw_split(plan.rest, panels, items) : 1, plan.blocks);
    else put(0, tiles(V, RES), 0, tiles(V, RES) * Nt, plan.tail.split > 0 ? plan.tail.split : 1, plan.blocks);
    if (!plan.wide) out9[4] = plan.tail.split > 0 ? plan.tail.rows * Nt : 0;
    return MRL_OK;
  }
  const bool fwd = launch == MRL_PROF_GEMM_FWD;
  const CutPlan plan = fwd ? plan_forward(chunk_rows, V, d) : plan_dh(chunk_rows, V, d, items);
  const int panels = (int)(round_up(V, 2 * BK) / BK), kind = cut_kind(plan.cuts, rows);
  const Cut cut = fwd ? cut_rows<MODE_FWD>(rows, kind) : cut_rows<MODE_DH>(rows, kind);
  const int all = cut.count() * (fwd ? tiles(V, RES) : Nt);
  put(cut.wide, cut.narrow, cut.half, all, !fwd && all % kRound > 0 ? dh_split(all % kRound, panels, items) : 1, plan.blocks);
  out9[8] = cut.start(cut.count() - 1);
  return MRL_OK;
}

extern "C" int mrl_diag_dw_tail_plan(int32_t V, int32_t d, int32_t* out12) {
  using namespace mrl;
  if (out12 == nullptr) return MRL_ERR_NULL;
  if (V <= 0 || d <= 0) return MRL_ERR_SHAPE;
  const int Mt = tiles(V, RES), Nt = tiles(d, RES);
  const SuperTile st = pick_super_tile(Nt);
  const DwTailPlan t = dw_tail_plan(Mt, Nt, st.m, st.n);
  out12[0] = t.m0; out12[1] = t.rows; out12[2] = t.split;
  for (int x = 0; x <= NXCD; ++x) out12[3 + x] = t.split > 0 ? t.first[x] : 0;
  return MRL_OK;
}
