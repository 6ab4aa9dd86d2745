// Internal kernel arguments and launchers (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vsd {

constexpr int kMaxL = 64;

struct SampleArgs {
  const void* X;             // [R, ld_d]
  const void* Y;             // [R, ld_t]
  const int32_t* d2t;        // [Vd] or null (identity)
  const int32_t* depth;      // [P*N] or null
  int32_t* tok_d;
  int32_t* tok_t;
  int32_t* tok_g;
  int32_t* err;
  int64_t R, ld_d, ld_t;
  int32_t L, Vd, Vt;
  float inv_tq, inv_tp;      // float(1/T)
  uint32_t k0, k1, offset;   // Philox key words and counter word 3
  // Fused sample + row statistics (all null for plain sampling):
  float* lse_q;              // [R]
  float* lse_p;              // [R] optional
  float* la;                 // [R,3]
  float* lq;                 // [R,3]
  // top-K renormalised KL term (fused only; kl_k > 0 turns it on)
  int32_t kl_k;
  int32_t* kl_idx;           // [R, kl_k]
  float* kl_grad;            // [R, kl_k]
  float* kl_row;             // [R]
  float kl_gscale;           // loss_scale * kl_weight / N / T_q
};

// One depth of a rollout with exact context (vsd_sample_step): path p's rows
// are X + p ld_d (along z~), Y + p ld_t (along z'), Yg + p ld_t (along
// z-bar); its tokens go to row p L + step of the token arrays.
struct SampleStepArgs {
  const void* X;
  const void* Y;
  const void* Yg;
  const int32_t* d2t;        // [Vd] or null
  const int32_t* depth;      // [paths] or null
  int32_t* tok_d;
  int32_t* tok_t;
  int32_t* tok_g;
  int32_t* err;
  int64_t paths, ld_d, ld_t;
  int32_t L, step, Vd, Vt;
  float inv_tq, inv_tp;
  uint32_t k0, k1, offset;
};

// Decode-time verification of the draft paths (vsd_verify_paths).
constexpr int64_t kPathsSplit = 128;  // most paths whose residual draw is split over workgroups
struct VerifyArgs {
  const void* X;             // [R, ld_d]
  const void* Y;             // [R, ld_t]
  const int32_t* inv;        // [Vt] draft index of target column t, -1 unmapped; null = identity
  const int32_t* depth;      // [paths] or null
  const float* la;           // [R, 3] log alpha of the three families (column 0: z~)
  const float* lse_q;        // [R]
  const float* lse_p;        // [R]
  int32_t* accept_len;       // [paths]
  int32_t* resample;         // [paths] target index, -1 when every token is kept
  unsigned long long* slot_best;  // [paths] zeroed result slots of a split draw, or null
  uint32_t* slot_done;       // [paths] zeroed counts of finished workgroups
  int32_t* err;
  int64_t paths, ld_d, ld_t;
  int32_t L, Vd, Vt;
  float inv_tq, inv_tp;
  uint32_t k0, k1, offset;
};

struct ScoreRowArgs {
  const void* X;
  const void* Y;
  const int32_t* d2t;
  const int32_t* depth;
  const int32_t* tok[3];     // draft, target, greedy
  float* lse_q;              // [R] optional
  float* lse_p;              // [R] optional
  float* la;                 // [R,3]
  float* lq;                 // [R,3]
  int32_t* err;
  int64_t R, ld_d, ld_t;
  int32_t L, Vd, Vt;
  float inv_tq, inv_tp;
  int32_t fam_lo, fam_hi;    // families [fam_lo, fam_hi) gathered on these rows (columns of la / lq)
  // top-K renormalised KL term (kl_k > 0 turns it on)
  int32_t kl_k;
  int32_t* kl_idx;           // [R, kl_k]
  float* kl_grad;            // [R, kl_k]
  float* kl_row;             // [R]
  float kl_gscale;           // loss_scale * kl_weight / N / T_q
};

// Columns of one block of a row, and the blocks from which a row's sum has 4
// groups of one segment and 4 groups of 4 (k_score.hip).
constexpr int kScoreBlockCols = 2048, kScoreGroups = 4, kScoreSegs16Blocks = 32;

// Wavefronts per row of k_score_rows.  A row is a serial chain of blocks (about 0.8 us each,
// load latency), so few rows want several wavefronts; many rows are bound by
// HBM, where a workgroup streaming one row beats four streaming one each (fewer
// DRAM pages open at a time).  With per-path depths many workgroups of a row
// each find it masked and leave (their launch takes longer than the pages
// save): many such rows go four to a workgroup, unless both vocabularies have
// segments for 16 wavefronts (then W = 16 is within 1 % of the best at any
// row count).  With the KL term every wavefront also seeds and compacts a
// top-K list, which only few rows repay.  us of vsd_score_paths, by W:
//                          rows     1       4      16    ragged 1      4      16
//   32k + 128k              256    68.8    29.5    29.4      68.1    29.4    27.5
//                           512    70.0    37.8    40.8      68.9    34.9    35.5
//                          1024   102.9    69.6    73.9      72.9    52.3    59.5
//                          2048   129.4   127.8   131.4     112.1    94.0   105.0
//                          4096   242.7   242.8   240.1     172.3   175.7   194.6
//                         16384   919.7   906.0   861.3     598.8   613.3   683.9
//                         65536  3567.3  3436.2  3351.6    2182.4  2390.7  2671.9
//   32k + 128k, float32     256    70.8    35.8    38.1      70.0    30.2    31.9
//                          1024   130.4   133.9   130.2     103.1    91.1    97.1
//                          2048   237.8   242.9   232.8     149.2   169.0   167.6
//                         16384  1779.6  1736.4  1699.1    1138.4  1199.7  1175.2
//   70k + 70k               256    63.0    26.6    23.7      62.2    26.6    21.9
//                          2048   113.8   113.1   108.8      94.7    80.3    79.2
//                         16384   810.0   784.0   741.5     533.8   543.0   537.5
//   32k + 128k, KL          256   103.9    42.4    37.7     100.6    42.6    37.6
//                           512   104.5    49.9    63.8     101.7    49.1    63.8
//                          2048   156.4   149.2   231.1     146.2   134.7   229.0
//                          4096   278.2   272.3   446.9     241.1   250.2   445.6
//   32k + 32k               256    35.4    19.2    26.5      33.2    19.4    26.8
//                          1024    41.5    36.7    52.9      40.1    32.4    48.9
//                          4096   109.6   106.4   175.7      74.6    75.7   164.0
//                         16384   384.9   361.5   633.3     258.1   261.0   621.8
//                         65536  1468.2  1391.7  2483.9     910.8   998.4  2429.5
//                        131072  2898.9  2779.1  4944.2    1762.2  1984.7  4869.4
//   32k + 32k, KL          1024    55.4    47.5   135.5      54.4    45.9   136.0
//                          2048    65.0    71.2   255.0      61.0    65.7   254.7
// Narrow rows around the line where W = 4 ends, W = 1 / W = 4 (in brackets one
// running sum per row, before rows were split):
//                         1024            1280            1536            1792            2048
//   32k + 32k         36.8 / 32.0     43.6 / 36.5     45.2 / 41.6     46.7 / 45.4     49.9 / 50.1   (50.0)
//   19k + 27k         30.1 / 26.4     35.3 / 29.6     36.4 / 33.4     37.8 / 36.8     39.1 / 39.6   (39.2)
//   9k + 9k           20.9 / 18.7     23.1 / 20.1     24.0 / 21.7     24.9 / 24.1     25.7 / 25.8   (25.7)
//   32k + 32k, f32    47.1 / 49.1     66.5 / 62.8     78.7 / 80.6     88.8 / 93.0     99.1 / 103.2  (99.8)
//   9k + 9k, f32      23.4 / 23.5     26.4 / 25.6     28.1 / 28.2     30.2 / 30.8     33.4 / 33.8   (33.6)
//   ragged, 32k + 32k 51.6 / 44.7     61.0 / 50.9                     65.3 / 62.6
//   the same, f32     53.2 / 56.8     61.4 / 66.1                     78.7 / 87.5
// A launch counts its work-items in 32 bits, and W = 16 takes 1024 a row: past
// 2^22 rows (over 500 GB of logits of 64k columns) rows go four to a workgroup.
constexpr int64_t kKlRowsW16 = 256, kKlRowsW4 = 1024;  // most rows with the KL term (W = 4: twice on wide rows)
constexpr int64_t kRaggedRowsW16 = 512, kRaggedBytesW4 = 4096;  // wide ragged rows; rows x element size
constexpr int64_t kNarrowBytesW4 = 3584;  // narrow rows x element size: W = 4 up to here and, full batches,
constexpr int64_t kNarrowRowsW1 = 8192;   // past this many rows
constexpr int64_t kMaxRowsW16 = ((int64_t)1 << 22) - 1;
inline int score_waves(int64_t R, int Vd, int Vt, int elem_bytes, bool kl, bool ragged) {
  const int longer = ((Vd > Vt ? Vd : Vt) + kScoreBlockCols - 1) / kScoreBlockCols;
  const int shorter = ((Vd < Vt ? Vd : Vt) + kScoreBlockCols - 1) / kScoreBlockCols;
  const bool wide = longer >= kScoreSegs16Blocks;
  if (wide && R <= kMaxRowsW16 &&
      (kl ? R <= kKlRowsW16 : !ragged || shorter >= kScoreSegs16Blocks || R <= kRaggedRowsW16))
    return 16;
  if (longer >= kScoreGroups && (kl     ? R <= (wide ? 2 : 1) * kKlRowsW4
                                 : wide ? R * elem_bytes <= kRaggedBytesW4
                                        : R * elem_bytes <= kNarrowBytesW4 || (!ragged && R > kNarrowRowsW1)))
    return 4;
  return 1;
}

struct CombineArgs {
  const float* la;           // [R,3]
  const float* lq;           // [R,3]
  const int32_t* depth;      // [P*N] or null
  float* survival;           // optional [R]
  float* ea;                 // optional [P*N]
  uint8_t* acc_flag;         // optional [R]
  uint8_t* val_flag;         // optional [R]
  float* o_prime;            // optional [R]
  float* beta;               // optional [R]
  float* zeta;               // optional [R]
  float* coef_a;             // [R]
  float* coef_b;             // [R]
  float* loss_pos;           // [P]
  int32_t* err;
  int32_t P, N, L;
  int32_t mode, car_input;
  float inv_tau;
  const float* kl_row;       // [R] KL row terms, or null (term off)
  float* kl_pos;             // optional [P]
  float kl_weight;
  float* loss_total;         // optional [1]
  float loss_scale;
  float w[kMaxL];            // w(l) = w_base^l, l = 1..L
};

struct BwdArgs {
  const void* X;
  void* G;
  const float* lse_q;
  const int32_t* tok_d;
  const int32_t* tok_t;
  const float* coef_a;       // [R], or null: a = 0
  const float* coef_b;       // [R], or null: b = 0
  int64_t R, ld;
  int32_t Vd;
  float inv_tq, scale;
  const int32_t* kl_idx;     // [R, kl_k] or null: sparse KL gradient terms added to the row
  const float* kl_grad;      // [R, kl_k]
  int32_t kl_k;
};

// ------------------------------------------------ fused LM-head variant ---
constexpr int kLmTile = 256;           // rows and vocabulary columns per logit tile
constexpr int kLmTilesPerSlice = 16;   // vocabulary tiles one forward workgroup walks

// Vocabulary slices of a V-column pass (a function of V only, so the float
// outputs of a row do not depend on the batch size).
inline int lm_nslice(int V) {
  const int tiles = (V + kLmTile - 1) / kLmTile;
  return (tiles + kLmTilesPerSlice - 1) / kLmTilesPerSlice;
}

// One slice's running state of one row (32 bytes).
struct LmPartial {
  float mraw, mc, s;   // log-sum-exp in shifted form
  float key;           // best Gumbel key
  int32_t idx;         // its draft index
  float gval;          // greedy maximum (target pass)
  int32_t gidx;
  int32_t pad;
};

// A forward over few row tiles is spread over the chip by single vocabulary
// tiles instead of slices: a workgroup then walks lm_run_tiles tiles, leaves
// every tile's state of every row and wavefront group in a region of the
// workspace, and k_lm_fold forms the slices' states from them in the order in
// which a workgroup that walks a slice does, so the results are the same.
constexpr int kLmCus = 256;                       // workgroups (one per CU) that run at a time
constexpr int64_t kLmTileBytesMax = 64ll << 20;   // largest such region
inline int lm_tiles(int V) { return (V + kLmTile - 1) / kLmTile; }

// Top-K renormalised KL term on the fused head: every row segment of the
// target pass keeps its few best mapped target logits; a slice's record
// holds the best kLmKlM of its four segments' lists and an upper bound of
// every value they dropped (-inf: none dropped).
constexpr int kLmKlM = 8;
struct LmKlEntry {
  float val;                 // raw target logit
  int32_t idx;               // its draft index
};

// A row the slice lists cannot decide is recomputed exactly over slices of
// the draft vocabulary, whose records (kLmRedoM entries each) take the place
// of the row's target-slice lists once the combine has read them: as many
// slices as fit there (at least one; the row's region is padded when one
// does not fit).
constexpr int kLmRedoM = 16;
inline int lm_redo_nslice(int Vd, int Vt) {
  const int tiles = (Vd + kLmTile - 1) / kLmTile;
  const int fit = lm_nslice(Vt) * kLmKlM / kLmRedoM;
  return fit < 1 ? 1 : fit < tiles ? fit : tiles;
}
// LmKlEntry records per row of the KL lists' region.
inline int lm_kl_stride(int Vd, int Vt) {
  const int lists = lm_nslice(Vt) * kLmKlM, redo = lm_redo_nslice(Vd, Vt) * kLmRedoM;
  return lists > redo ? lists : redo;
}

// Bytes of the tiles' states.
inline size_t lm_tile_bytes(int64_t R, int Vd, int Vt) {
  return (size_t)R * (size_t)(lm_tiles(Vd) + lm_tiles(Vt)) * 2 * sizeof(LmPartial);
}
// Tiles a workgroup walks: the fewest with which every run has a CU at once, or
// 0: that takes more than 14 tiles, so the slices (16 of them) keep the CUs about
// as busy, or the region would be too large.  Where it ends depends on both
// vocabularies: past 1280 rows for 32k + 128k, 3584 for 32k + 32k, 21 760
// for 1000 + 5000.  A run's length needs no other size: its tiles' states are 64
// bytes a row against H products a column, and the rule is never slower than the
// slices from H = 64 on.  us of scoring given paths by slices / by runs:
//                  rows     16           192          512          1008         1248         3072         6144
//   32k + 128k
//     H = 4096        1156 / 334   1203 / 373   1227 / 621   1366 / 1102  1517 / 1389
//     H = 512          253 / 86     251 / 90     253 / 135    263 / 210    279 / 265
//     H = 64           145 / 60     138 / 65     139 / 83     141 / 117    146 / 139
//   32k + 32k
//     H = 4096        1135 / 147   1189 / 171   1201 / 277   1199 / 485   1193 / 580   1481 / 1334
//     H = 64           137 / 38     130 / 41     130 / 52     132 / 69     134 / 76     140 / 134
//   8k + 16k
//     H = 1024         370 / 55     366 / 58     368 / 63     370 / 89     371 / 95     377 / 184    442 / 355
//   1000 + 5000
//     H = 4096         708 / 109    709 / 111    712 / 114    716 / 118    717 / 124    741 / 218    788 / 357
//     H = 64            85 / 30      85 / 32      85 / 32      86 / 33      86 / 34      89 / 45      95 / 59
//   256 + 300
//     H = 64            24 / 23      26 / 25      26 / 25      29 / 26      27 / 26      30 / 29      34 / 34
// The same with the KL term (K = 10), where a slice's 16 tiles in a row are also
// 16 epilogues of list insertions (by slices it took up to 1.5 times as long as
// with the epilogue that gave a row four threads instead of two):
//                  rows     16           256          640          1536
//   32k + 128k
//     H = 4096        1590 / 456   1660 / 515   1618 / 1052
//     H = 256          550 / 193    560 / 191    552 / 341
//   44k + 44k
//     H = 4096        1578 / 352   1720 / 378   1670 / 716   1703 / 1260
//     H = 256          557 / 169    637 / 169    638 / 285    645 / 434
//   5000 + 5000
//     H = 4096        3428 / 201   3893 / 199   4022 / 205   4259 / 237
//     H = 256          797 / 104   1476 / 98    1475 / 99    1650 / 108
// (a run of 14 on 1536 rows of 32k + 128k, two rounds: 1695 / 2581 at H = 4096.)
constexpr int kLmRunMost = 14;
inline int lm_run_tiles(int64_t R, int Vd, int Vt) {
  const int64_t row_tiles = (R + kLmTile - 1) / kLmTile;
  if ((int64_t)lm_tile_bytes(R, Vd, Vt) > kLmTileBytesMax) return 0;
  for (int run = 1; run <= kLmRunMost; ++run)
    if (row_tiles * ((lm_tiles(Vd) + run - 1) / run + (lm_tiles(Vt) + run - 1) / run) <= kLmCus) return run;
  return 0;
}

// Runs of a pass over V columns.
inline int lm_runs(int V, int run_tiles) { return (lm_tiles(V) + run_tiles - 1) / run_tiles; }
// Bytes of the KL term's lists by runs: a record of kLmKlM entries and a bound
// per row and run.
inline size_t lm_run_list_bytes(int64_t R, int runs_t) {
  return (size_t)R * (size_t)runs_t * (kLmKlM * sizeof(LmKlEntry) + sizeof(float));
}

struct LmFwdArgs {
  const void* Hd;            // [R, H] bf16
  const void* Ht;            // [R, H] bf16
  const void* Wd;            // [Vd, H] bf16
  const void* Wt;            // [Vt, H] bf16
  const int32_t* inv;        // [Vt] draft index of each target column (-1: none); null = identity
  LmPartial* part;           // [R, nslice_t + nslice_d], target slices first
  LmKlEntry* kl_part;        // KL term: [R, kl_stride] rows of kl_lists lists of kLmKlM, or null
                             // (term off)
  float* kl_bound;           // KL term: [R, kl_lists] bound of the dropped values
  int32_t kl_lists;          // KL term: lists per row, one per target slice (with tile_part, run)
  LmPartial* tile_part;      // null, or [tiles_t + tiles_d, 2, R] states of single tiles
  int32_t run_tiles;         // tiles a workgroup walks with tile_part
  int64_t R;
  int32_t kl_stride;         // KL term: LmKlEntry records per row of kl_part
  int32_t H, Vd, Vt;
  int32_t nslice_t, nslice_d;
  int32_t sample;            // 0: log-sum-exp only (scoring given tokens)
  float inv_tq, inv_tp;
  uint32_t k0, k1, offset;
};

struct LmCombineArgs {
  const LmPartial* part;
  const void* Hd;
  const void* Ht;
  const void* Wd;
  const void* Wt;
  const int32_t* d2t;
  const int32_t* depth;
  const int32_t* tok_in[3];  // scoring: given tokens; sampling: null
  int32_t* tok_out[3];       // sampling: drawn tokens
  float* lse_q;
  float* lse_p;              // optional
  float* la;                 // [R,3]
  float* lq;                 // [R,3]
  int32_t* err;
  int64_t R;
  int32_t L, H, Vd, Vt;
  int32_t nslice_t, nslice_d;
  float inv_tq, inv_tp;
  // top-K renormalised KL term (kl_k > 0 turns it on)
  int32_t kl_k;
  const LmKlEntry* kl_in;    // [R, kl_in_stride]: the forward's kl_lists lists
  int32_t kl_in_stride, kl_lists;
  const float* kl_bound;     // [R, kl_lists]
  LmKlEntry* kl_part;        // [R, kl_stride]: the recompute's kl_nslice records of kLmRedoM (slice
                             // lists lie there too, and are read before)
  int32_t kl_stride;         // lm_kl_stride(Vd, Vt)
  int32_t* kl_count;         // [1] rows the lists could not decide (reset before the combine)
  int32_t* kl_list;          // [R] those rows, in the order they were found
  int32_t kl_nslice;         // lm_redo_nslice(Vd, Vt)
  int32_t* kl_idx;           // [R, kl_k]
  float* kl_grad;            // [R, kl_k]
  float* kl_row;             // [R]
  float kl_gscale;           // loss_scale * kl_weight / N / T_q
};

struct LmBwdArgs {
  const void* Hd;
  const void* Wd;
  void* G;                   // [R, ldg] bf16: gradient w.r.t. the draft logits
  void* dH;                  // [R, H] bf16
  float* dW;                 // [Vd, H] fp32 or null: gradient w.r.t. the draft head's weight
  const float* lse_q;
  const int32_t* tok_d;
  const int32_t* tok_t;
  const float* coef_a;
  const float* coef_b;
  const int32_t* kl_idx;     // [R, kl_k] or null: the KL term's sparse gradient, added to G
  const float* kl_grad;      // [R, kl_k]
  int32_t kl_k;
  int64_t R, ldg;
  int32_t H, Vd;
  float inv_tq, scale;
};

// C = A^T B with A [K, M] and B [K, N] row-major bf16, C [M, N] fp32.
struct LmGemmTNArgs {
  const void* A;
  const void* B;
  float* C;
  int64_t M, lda;
  int64_t ldb, ldc;
  int32_t N, K;
};

struct LmGemmNNArgs {
  const void* A;             // [M, K] bf16
  const void* B;             // [K, N] bf16
  void* C;                   // [M, N] bf16
  int64_t M, lda;
  int64_t ldb, ldc;
  int32_t N, K;
};

// Bytes from the start of four consecutive rows of a bf16 matrix [*, n] with row
// stride ld that a load of them may touch: up to the last row's n columns (in
// whole 16-byte chunks, which a row's 16-byte alignment keeps within its last
// column's chunk).  The stride beyond them is not the matrix's: with a gradient
// buffer that is a column range of a wider one, the last row's lies past the
// allocation.
constexpr uint32_t lm_kmajor_bytes(int64_t ld, int n) { return (uint32_t)((3 * ld + ((n + 7) & ~7)) * 2); }

// the inverse map; the launch also clears `nclear` words at `clear`
hipError_t launch_lm_inv(const int32_t* d2t, int Vd, int Vt, int32_t* inv, int32_t* err, uint32_t* clear, int nclear,
                         hipStream_t s);
hipError_t launch_lm_fwd(const LmFwdArgs& a, hipStream_t s);
hipError_t launch_lm_combine(const LmCombineArgs& a, hipStream_t s);
hipError_t launch_lm_kl_reset(const LmCombineArgs& a, hipStream_t s);
hipError_t launch_lm_kl_redo(const LmCombineArgs& a, hipStream_t s);
hipError_t launch_lm_bwd(const LmBwdArgs& a, hipStream_t s);

hipError_t launch_sample(const SampleArgs& a, bool bf16, hipStream_t s);
hipError_t launch_sample_step(const SampleStepArgs& a, bool bf16, hipStream_t s);
hipError_t launch_verify(const VerifyArgs& a, bool bf16, hipStream_t s);
hipError_t launch_score_rows(const ScoreRowArgs& a, bool bf16, hipStream_t s);
// the per-position combine and, if asked for, the loss total
hipError_t launch_combine(const CombineArgs& a, hipStream_t s);
hipError_t launch_bwd(const BwdArgs& a, bool bf16, hipStream_t s);

}  // namespace vsd
