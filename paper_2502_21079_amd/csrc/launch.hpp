// Internal launch interface between the C ABI (api.hip) and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace adaspa {

typedef uint16_t u16;

// Every row of every pattern, only the rows that the key-split kernel is to
// take (split_rows), only the others.
enum { PICK_ALL = 0, PICK_SPLIT = 1, PICK_OTHERS = 2 };

struct AttnParams {
  const u16* q;
  const u16* k;
  const u16* v;
  u16* o;
  float* lse;                 // may be null
  const int32_t* row_ptr;     // sparse only
  const int32_t* col_idx;     // sparse only
  int64_t col_count;          // entries readable in col_idx (sparse only)
  int batch_heads;            // B * H
  int seqlen;
  int block;                  // sparse block size
  int nkb;                    // key blocks (sparse)
  int nqt;                    // query tiles per head (set by the launcher)
  int n_wg;                   // workgroups (set by the launcher)
  float scale;
  float scale_log2;           // scale * log2(e)
  int tq0, tq1;               // sparse: text query blocks [tq0, tq1), dispatched first
  int kb_guess, n_guess;      // sparse: first text block and the text block count (-1, 0: none),
                              // whose tiles every row begins with under the text sink
  bool split;                 // the key-split kernel takes the problem (use_key_split)
  int n_tail;                 // the last 256-row items that run key-split (split_tail): dense, and
                              // sparse patterns that keep every block
  int pick;                   // sparse: which rows a launch runs (PICK_*, set by the launcher)
  int ends;                   // sparse: tiles at each end of the sequence that come first when the
                              // call names no text range (set by the launcher)
  int64_t pick_entries;       // sparse: with PICK_*, the most entries of a pattern that runs key-split
  uint32_t* claim;            // 9 work-queue counters (one per XCD + a flag), or null
  int n_items;                // work items: (head, query tile) or (head, query block / pair)
  int n_static;               // sparse: items [0, n_static) run in the static order
  // Single-pass search only: log2 of each row's mass in each key block,
  // [B*H, nkb, L], and log2 e * LSE of each row, [B*H, L] (scratch), and the
  // block masses W, [B*H, nkb, nkb].
  float* ylog;
  float* ylse2;
  float* wmass;
};

// Whether attention over batch_heads sequences of length seqlen runs in the
// key-split kernel (64 query rows per workgroup): by the shape alone, so that
// every entry point takes a problem the same way and their results agree bit
// for bit.  512 such workgroups run in two rounds on 256 CUs; up to there the
// key split is the faster one (8,192 tokens, dense, us, one-tile-per-step
// kernels against key split: 2 heads = 256 workgroups 113 -> 48 at d 64 and
// 154 -> 83 at d 128; 4 heads = 512 workgroups 114 -> 92 and 160 -> 159; but 6
// heads 132 -> 136 and 193 -> 239).
constexpr int64_t kSplitMaxTiles = 512;
inline bool use_key_split(int64_t batch_heads, int seqlen) {
  return batch_heads * ((seqlen + 63) / 64) <= kSplitMaxTiles;
}

// Beyond that, dense attention runs (head, 256-row tile) items, 256 at a time
// at d 128 (one workgroup per CU); at d 64 an item is two workgroups of 128
// rows, three of which share a CU, so up to 384 run at a time.  When the items
// come to a few more than a multiple of 256, those few run key-split instead,
// four workgroups each: the number of such items, always the last ones.
// Dense, us, without and with it:
// - d 128, where they are a last round of their own: 8,192 tokens x 9 heads (one
//   round and 32 items) 358 -> 284, x 10 (and 64) 359 -> 297, 16,384 x 5 (and
//   64) 706 -> 577, 35,000 x 4 (two and 36) 2410 -> 2095, 8,192 x 33 (four and
//   32) 985 -> 941; after many rounds the CUs no longer end together and the
//   last items hide among the others' ends, 110,336 x 3 (five and 13) gained
//   nothing, so this stops at four;
// - d 64, where they make CUs hold one workgroup more than others for their
//   whole time: 8,192 x 9 177 -> 173, 35,000 x 4 1275 -> 1239, 16,384 x 13 (three
//   and 64) 852 -> 836.  Below 8,192 tokens the second launch costs more
//   (4,096 x 17 90.4 -> 91.6), and 65 to 128 items are slower at every length
//   (8,192 x 12 198 -> 220, 35,000 x 8 2351 -> 2475).
inline int split_tail(int64_t batch_heads, int seqlen, int head_dim) {
  const int64_t n = batch_heads * ((seqlen + 255) / 256), rest = n % 256;
  if (use_key_split(batch_heads, seqlen) || n < 256 || n / 256 > 4) return 0;
  if (head_dim == 64 && seqlen < 8192) return 0;
  return rest <= 64 ? (int)rest : 0;
}

struct MassParams {
  const u16* q;
  const u16* k;
  const float* lse;
  float* w;                   // [B*H, nkb, nkb]
  int batch_heads;
  int seqlen;
  int block;
  int nkb;
  int n_wg;
  float scale_log2;
  uint32_t* claim;            // 8 work-queue counters (one per XCD), or null
  int n_items;                // work items (set by the launcher): n_whole (head, query-block group)
  int n_whole, n_split;       // items over all key blocks, then n_split ranges of each other one
};

constexpr int kMaxHeads = 512;
constexpr int kMaxBlocks = 8192;

// Rows whose masses one workgroup of the coverage curve adds up.  Up to
// kWaveBlocks blocks a wave sorts a row: four waves, each one to sixteen rows,
// few enough for four workgroups per CU, and at most 64, so that the partial
// curves to be added up stay few.  Longer rows are sorted by the whole workgroup
// one after another, so one or two each (one row of curves per row of masses,
// 2,582 blocks x 1 head 399 us, with two 464, with four 481; x 12 heads 3677,
// 3535 and 5703).
constexpr int kWaveBlocks = 2048;
inline int select_rows_per_wg(int rows, int nb) {
  if (nb > kWaveBlocks) return rows >= 8192 ? 2 : 1;
  const int per_wave = rows / 4096;
  return 4 * (per_wave < 1 ? 1 : (per_wave > 16 ? 16 : per_wave));
}

struct SelectParams {
  const float* w;             // [R, nb] masses, R = B*H*nb rows
  int32_t* row_ptr;
  int32_t* col_idx;
  int32_t* head_k_out;        // may be null
  float* head_recall_out;     // may be null
  // workspace
  int64_t* ws_sums;           // exact sums between the kernels: two per row (TOPK), partial curves
                              // [B*H, n_parts, nb] (COVERAGE), [B*H, n_parts, 4] (HIERARCHICAL)
  int32_t* ws_headk;          // [B*H]
  int32_t* ws_base;           // [B*H] first col_idx entry of each head (many heads only)
  int rows_per_wg, n_parts;   // COVERAGE: rows of one partial curve; parts per head (also HIERARCHICAL)
  int base_ready;             // ws_base holds the heads' first entries
  int summed;                 // COVERAGE: the first partial curve of a head holds the sum of all
                              // (rows_per_wg to summed are set by the launcher)
  int batch_heads;
  int heads;
  int nb;
  int text_lo, text_hi;       // text block range [lo, hi]; lo > hi when none
  int kmin;                   // smallest allowed count, max(1, #text blocks)
  int mode;                   // 0 = TOPK, 1 = COVERAGE, 2 = HIERARCHICAL
  int k_base, k_hi, k_lo;     // HIERARCHICAL: counts at s, (1+s)/2 and (3s-1)/2
  int recall_thr_bp;          // HIERARCHICAL: Recall threshold
  int64_t cap;                // Q32 cap = floor(2^62 / (nb*nb))
  int32_t head_param[kMaxHeads];  // TOPK: k_h; COVERAGE: tau_bp
};

hipError_t launch_dense(AttnParams a, int head_dim, hipStream_t st);
hipError_t launch_sparse(AttnParams a, int head_dim, hipStream_t st);
hipError_t launch_block_mass(MassParams a, int head_dim, hipStream_t st);
// Dense attention + LSE and the block masses of the same rows: one kernel, or
// where a.split or a.n_tail the dense launches and then the mass pass (m.lse is
// a.lse then, and unused otherwise).  a.claim: the optional work-queue counters.
hipError_t launch_fused_search(AttnParams a, MassParams m, int head_dim, hipStream_t st);
// Dense attention + LSE and the block masses of its LSE in one pass over
// Q K^T (a.ylog, a.ylse2: scratch of B*H*nkb*L and B*H*L floats; a.wmass:
// the masses), then the masses summed from the scratch.
hipError_t launch_single_pass_search(AttnParams a, int head_dim, hipStream_t st);
hipError_t launch_select(SelectParams p, hipStream_t st);

}  // namespace adaspa
