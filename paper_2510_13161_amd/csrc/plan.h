// Launch planning of a verify pass, on the host: the GEMMs' shapes and the
// workspace layout. No HIP calls, so the same code runs where there is no GPU.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "kernels.h"
#include "msd.h"

namespace msd {

// Scratch of msd_verify_block_static: MSD_STATIC_SCRATCH_BYTES for a block's
// workspace without the GEMMs' split partials and counters, and room for
// those: at most 72 MiB of partials (two workgroups on each of 256 compute
// units, 4 tiles of 9 row tiles each) and a few KB of counters. With the partials
// inside the first bound, a block that just fits would have to run other
// shapes, and so sum in another order, than in a caller's workspace.
constexpr size_t kStaticSplitBytes = (size_t)73 << 20;
constexpr size_t kStaticScratchBytes = MSD_STATIC_SCRATCH_BYTES + kStaticSplitBytes;

struct GemmShape {
  int n_tiles, K, splits, waves, jt;
  int wg_tiles = 1;
  int row_groups = 0;
  int split_from = 0;
};

struct Shapes {
  GemmShape qkv, o, up, down, head;
};

// The GEMMs of a block of mt row tiles, and what the workspace keeps for them:
// the most that any block of 1 .. mt row tiles uses, as split counts and tile
// widths go up and down with the row tiles and a workspace sized for a program's
// largest block has to serve its smaller ones.
struct RowPlan {
  Shapes s;
  size_t part_bytes;       // split partials
  int32_t split_tiles;     // split-K counters
  int32_t head_tiles;      // column tiles of the head
};

// What a plan depends on besides the block: the model, its device and the
// launch-shape overrides; and the plans of all row tile counts (plan_rows).
struct PlanInputs {
  msd_model_config cfg;
  int32_t n_cus = 256;             // compute units of the model's device
  int32_t target_wgs = 0;          // > 0: split-K sized for about this many workgroups
  int32_t waves = 8;               // waves of a split-K workgroup for one row tile
  int32_t qkv_jt = 2;              // 16-column sub-tiles of the QKV projection's tiles at one row tile (2 or 4)
  int32_t rows_max_splits = 4;     // its splits of K at most
  int32_t rows_min_tiles = 256;    // 64-column tiles of a GEMM that takes the LDS-shared kernel
  int32_t rows_min_mt = 3;         // row tiles from which it does
  bool rows_forced = false;        // MSD_ROWS_MIN_TILES set: no balance check
  int32_t rows_narrow = 1;         // narrow GEMMs: many splits, deferred epilogue, or row groups
                                   // (0 off, 1 by weights, 2 many splits at any size)
  int32_t rows_narrow_mt = 3;      // row tiles from which it does
  RowPlan rows[kMaxMT];            // of mt = 1 .. kMaxMT row tiles, at mt - 1
};

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// 16-row tiles of M rows, 1 .. kMaxMT (a block of more rows goes through no
// GEMM). From 4 on every product of a padding tile would be matrix-core time and
// power that the rows in use lack: at 7 tiles instead of 9 (99 rows) the 14B
// gate+up takes 100 -> 82 us, at 4 instead of 5 (63 rows) 72 -> 63.
inline int row_tiles(int64_t M) { return (int)std::min<int64_t>((M + 15) / 16, kMaxMT); }

// Split-K factor. A workgroup streams its 1/s of a tile at about one
// compute unit's rate, so a GEMM lasts as long as its busiest unit: W =
// n_tiles * s workgroups over C units put ceil(W / C) of them on one unit.
// s maximises the balance W / (C ceil(W / C)) (the smallest s on a tie),
// with W <= per_cu * C (more would wait for a second dispatch round; per_cu
// is how many of these workgroups a unit holds) unless s = 1, and at least
// 2 k-steps per wave. Measured: 66B tree, O and down projections (144
// tiles, 4-wave workgroups, two a unit) 2 -> 3 splits: 59.4 -> 46.4 us and
// 207.6 -> 154.2 us. m->target_wgs > 0 instead asks for about that many
// workgroups (tuning).
inline int splits_for(const PlanInputs* m, int n_tiles, int K, int waves, int per_cu) {
  const int ks = K / 32;
  int max_s = ks / (2 * waves);
  if (max_s < 1) max_s = 1;
  if (m->target_wgs > 0) {
    const int want = std::max(1, (m->target_wgs + n_tiles / 2) / n_tiles);
    return want < max_s ? want : max_s;
  }
  const int64_t C = m->n_cus;
  int best = 1;
  double best_bal = 0.0;
  for (int s = 1; s <= max_s; ++s) {
    const int64_t W = (int64_t)n_tiles * s;
    if (s > 1 && W > (int64_t)per_cu * C) break;
    const double bal = (double)W / (double)(C * ((W + C - 1) / C));
    if (bal > best_bal + 1e-9) {
      best = s;
      best_bal = bal;
    }
  }
  return best;
}

// Several row tiles, wide GEMMs (256 or more 64-column tiles): 4 tiles a
// workgroup sharing the activation through LDS (one workgroup per compute
// unit from 4 row tiles on, by its LDS ring and registers; two up to 3).
// Splits of K as for split-K above, for the best balance of
// ceil(n_tiles / 4) * s workgroups over the units within two workgroups a unit
// (one dispatch round, or two from 4 row tiles on: 66B FFN up, 144 workgroup
// tiles in 3 splits instead of whole K, two layers at 99 rows 1284 -> 1189 us,
// at 144 1456 -> 1365, at 66 997 -> 945), at most m->rows_max_splits (each split adds an fp32 partial of the
// whole [M][64] tile to write and read back) and at least 8 k-steps a
// split. Returns 0 where at 3 row tiles no split count balances at least 3/4
// of the units (then the split-K kernel runs), unless the kernel is forced;
// from 4 row tiles on sharing the activation gains more than the balance (66B
// FFN up, 144 workgroup tiles, whole K: 215 -> 165 us at 80 rows, 342 -> 229
// at 144). Measured:
// 14B batch 16, FFN up (108 workgroup tiles, 2 splits) and LM head (594,
// whole K): 136.8 -> 97.0 us and 740 -> 522 us; 66B tree (3 row tiles, one
// workgroup a unit then): QKV (108, 2 splits) 118.3 -> 97.2 us, LM head
// (197) 224.8 -> 166.5 us, its FFN up (144 workgroup tiles: 0.56 at best)
// 168.8 -> 177.7 us.
inline int rows_splits(const PlanInputs* m, int n_tiles, int K, int per_cu) {
  const int64_t C = m->n_cus;
  const int64_t wg = (n_tiles + 3) / 4;
  const int max_s = std::max(1, std::min(m->rows_max_splits, (K / 32) / 8));
  int best = 1;
  double best_bal = 0.0;
  for (int s = 1; s <= max_s; ++s) {
    const int64_t W = wg * s;
    if (s > 1 && W > 2 * C) break;
    const double bal = (double)W / (double)(C * ((W + C - 1) / C));
    if (bal > best_bal + 1e-9) {
      best = s;
      best_bal = bal;
    }
  }
  if (best_bal >= 0.75 || m->rows_forced) return best;
  return per_cu > 1 ? 0 : best;
}

// Narrow GEMMs (fewer tiles than m->rows_min_tiles) from 3 row tiles on:
// the same kernel with many splits of K, so that the 144-row MFMA work
// spreads over the chip, and the split sum plus epilogue in a kernel of its
// own (gemm_epi_kernel) instead of in the last split to arrive; the split
// count as above, at most kRowsNarrowSplits. m->rows_narrow: 0 off, 1 at 3
// row tiles for matrices of at least kRowsNarrowMinWeights weights (each
// split writes and the epilogue kernel reads an fp32 partial of all M rows)
// and from 4 row tiles for all that row groups (below) leave, 2 any size
// (tests). Measured against the split-K kernel's last-arrival epilogue (us,
// both kernels): 14B at 144 rows QKV 51.7 -> 43, O 35.5 -> 29.8, FFN down 66.4
// -> 50; 99 rows O 34.6 -> 27.1; at 3 row tiles O (26M weights, 36 rows) 20.8
// against 19.5, so not there; 66B tree (3 row tiles, two workgroups a unit, 7
// splits) O 46.4 -> 37.4, down 154.2 -> 121; at 2 row tiles slower (14B tree,
// QKV 24.3 against 22.4).
constexpr int kRowsNarrowSplits = 16;
constexpr int64_t kRowsNarrowMinWeights = 32ll << 20;
inline int rows_narrow_splits(const PlanInputs* m, int n_tiles, int K, int per_cu) {
  const int64_t C = m->n_cus;
  const int64_t wg = (n_tiles + 3) / 4;
  const int max_s = std::max(1, std::min(kRowsNarrowSplits, (K / 32) / 8));
  int best = 1;
  double best_bal = 0.0;
  for (int s = 1; s <= max_s; ++s) {
    const int64_t W = wg * s;
    if (s > 1 && W > per_cu * C) break;
    const double bal = (double)W / (double)(C * ((W + C - 1) / C));
    if (bal > best_bal + 1e-9) {
      best = s;
      best_bal = bal;
    }
  }
  return best;
}

// Wide GEMMs of more workgroups than one dispatch round takes (the LM head):
// the rounds that are full run whole K, the workgroups of the last one are
// split in K so that they fill it too (14B vocabulary: 594 workgroups, 82 in the
// last round; head with top-4 at 144 rows 540-547 -> 470 us). s: their splits,
// returned: the first tile of the last round, 0 where there is nothing to gain.
inline int rows_tail(const PlanInputs* m, int n_tiles, int K, int per_cu, int* s) {
  const int slots = m->n_cus * per_cu, wg = (n_tiles + 3) / 4;
  const int full = wg / slots * slots, last = wg - full;
  if (full == 0 || last == 0) return 0;
  *s = std::min(std::min(slots / last, kRowsNarrowSplits), K / 32 / 8);
  return *s > 1 ? 4 * full : 0;
}

// Small matrices at several row tiles (fewer than m->rows_min_tiles 64-column
// tiles): the row tiles in groups of at most 3, whole K, as many groups as fit
// the compute units. Split-K and the LDS-shared kernel spend their time there on
// partials and hand-offs (0.6B-shaped layer at 72 rows: 18 us a GEMM, 11.5 in
// groups). The line by weights: from 4 row tiles 24M (21M weights in 64 tiles
// at 144 rows 32.5 us against 36.5 in the LDS-shared kernel with 16 splits, 63
// rows 25.1 against 27.0; 26M in 80 tiles 30.9 against 29.7 and 26.6 against
// 23.7), at 2 and 3 row tiles 8M (6M: 10.7 against 12.8 us; 21M: 25.5 against
// 17.3), and there not the residual projections, whose K is the longer one
// and whose split-K hand-off is a single row tile a wave (3M at 2 row tiles:
// 15.1 against 12.4).
constexpr int64_t kGroupMaxWeights = 24ll << 20, kGroupMaxWeightsFewRows = 8ll << 20;
inline int row_groups(const PlanInputs* m, int n_tiles, int mt) {
  return std::min(mt, std::max((mt + 2) / 3, m->n_cus / n_tiles));
}

// Tiles and waves per workgroup. With one row tile, a GEMM with fewer
// 64-column tiles than the workgroup target runs split-K workgroups of
// m->waves (8) waves, one with more (the LM head) whole-K workgroups of 4
// waves; 2 and 3 row tiles 64-column tiles of 4 waves, unless in row groups or in
// the kernel that shares the activation through LDS; from 4 row tiles on one of
// these two. The SwiGLU FFN up projection with up to 3 row tiles: whole-K
// 128-column tiles of 2 waves (216 workgroups at the 14B shape, one dispatch
// round: at most one per CU), at one row tile only where its 64-column tiles
// do not fit the compute units (else split-K tiles of 8 waves: 6M weights 10.4
// -> 8.8 us), at 3 only where the LDS-shared kernel does not balance (14B, 36
// rows: 63 -> 59 us there).
// A function of the row tiles alone: kappa, the cache's capacity and the memory
// that a caller has change neither the kernels that a block of so many rows runs
// nor the order of its sums.
inline Shapes shapes(const PlanInputs* m, int mt) {
  const msd_model_config& c = m->cfg;
  const bool one = mt == 1;
  Shapes s;
  s.qkv.n_tiles = (c.n_heads + 2 * c.n_kv_heads) * c.head_dim / kTileN;
  s.qkv.K = c.d_model;
  s.o.n_tiles = c.d_model / kTileN;
  s.o.K = c.n_heads * c.head_dim;
  s.up.n_tiles = c.act == MSD_ACT_SWIGLU ? c.d_ffn / 32 : c.d_ffn / kTileN;
  s.up.K = c.d_model;
  s.down.n_tiles = c.d_model / kTileN;
  s.down.K = c.d_ffn;
  s.head.n_tiles = (c.vocab + kTileN - 1) / kTileN;
  s.head.K = c.d_model;
  for (GemmShape* g : {&s.qkv, &s.o, &s.up, &s.down, &s.head}) {
    g->jt = 4;
    g->waves = one && g->n_tiles < m->n_cus ? m->waves : 4;
  }
  // The QKV projection at one row tile, where twice its 64-column tile count
  // still fits the compute units: 32-column tiles (16 rotary pairs of a head)
  // of 8 waves, whole K (no split hand-off), 224 workgroups at the 14B
  // shape. Measured at the 14B chain: 18.82 -> 18.06 us per launch against
  // 64-column tiles with 2 splits of K.
  if (one && m->qkv_jt == 2 && 2 * s.qkv.n_tiles <= m->n_cus) {
    s.qkv.jt = 2;
    s.qkv.n_tiles = (c.n_heads + 2 * c.n_kv_heads) * c.head_dim / 32;
    s.qkv.waves = 8;
  }
  // the LM head at one row tile: 128-column tiles of 4 waves, unless its
  // 64-column tiles fit the compute units (split-K tiles of 8 waves as the
  // projections': 4096 x 5120 weights 36.7 -> 16.3 us, 4096 x 1024 14.1 -> 9.5)
  if (one && s.head.n_tiles >= m->n_cus) {
    s.head.jt = 8;
    s.head.n_tiles = (c.vocab + 2 * kTileN - 1) / (2 * kTileN);
    s.head.waves = 4;
  }
  for (GemmShape* g : {&s.qkv, &s.o, &s.up, &s.down, &s.head}) {
    const int64_t weights = (int64_t)g->n_tiles * kTileN * g->K;
    const bool wide = g->n_tiles >= m->rows_min_tiles, resid = g == &s.o || g == &s.down;
    const int per_cu = mt <= 3 ? 2 : 1;
    if (!one && !wide && m->rows_narrow == 1 &&
        (mt >= 4 ? weights <= kGroupMaxWeights
                 : weights <= kGroupMaxWeightsFewRows && !resid)) {
      g->row_groups = row_groups(m, g->n_tiles, mt);
      g->waves = 8;
      g->splits = 1;
      continue;
    }
    int rs = 0;  // splits of the LDS-shared kernel (4 tiles a workgroup); 0: not taken
    const bool pair_up = g == &s.up && c.act == MSD_ACT_SWIGLU && mt <= 3 && !(one && g->n_tiles <= m->n_cus);
    if (g->jt == 4 && wide && mt >= m->rows_min_mt)
      rs = rows_splits(m, g->n_tiles, g->K, per_cu);
    else if (g->jt == 4 && !wide && !pair_up && mt >= m->rows_narrow_mt &&
             (m->rows_narrow == 2 || (m->rows_narrow == 1 && (mt >= 4 || weights >= kRowsNarrowMinWeights))))
      rs = rows_narrow_splits(m, g->n_tiles, g->K, per_cu);
    if (rs > 0) {
      g->wg_tiles = 4;
      g->waves = 4;
      g->splits = rs;
      int tail = 0;
      if (rs == 1) g->split_from = rows_tail(m, g->n_tiles, g->K, per_cu, &tail);
      if (g->split_from > 0) g->splits = tail;
      continue;
    }
    if (mt >= 4) {  // the LDS-shared kernel switched off
      g->row_groups = row_groups(m, g->n_tiles, mt);
      g->waves = 8;
      g->splits = 1;
      continue;
    }
    if (pair_up) {
      g->jt = 8;
      g->n_tiles = c.d_ffn / 64;
      g->waves = 2;
    }
    g->splits = splits_for(m, g->n_tiles, g->K, g->waves, g->waves >= 8 ? 1 : 2);
  }
  return s;
}

// Fills m->rows from the rest of *m: once per model.
inline void plan_rows(PlanInputs* m) {
  RowPlan most{};
  for (int mt = 1; mt <= kMaxMT; ++mt) {
    most.s = shapes(m, mt);
    for (const GemmShape* g : {&most.s.qkv, &most.s.o, &most.s.up, &most.s.down, &most.s.head}) {
      if (g->splits <= 1) continue;
      const size_t part = (size_t)(g->n_tiles - g->split_from) * g->splits * mt * g->jt * 256 * sizeof(float);
      most.part_bytes = std::max(most.part_bytes, part);
      most.split_tiles = std::max(most.split_tiles, g->n_tiles);
    }
    most.head_tiles = std::max(most.head_tiles, most.s.head.n_tiles);
    m->rows[mt - 1] = most;
  }
}

struct Layout {
  Shapes s;
  size_t x, stats, q, img_x, img_h, img_f, img_attn, img_act, partial, counters, part_o, part_ml,
      tile_ms, tile_top, head_ms, head_top, total;
  size_t split_bytes;  // of total: split partials past the attention's, and their counters
  int64_t n_counters, n_gemm_counters;
  int32_t MT, max_chunks;
};

// image bytes of an [M][K] activation
inline size_t img_bytes(int K, int MT) { return (size_t)(K / 32) * MT * 1024 * sizeof(uint16_t); }

// The workspace of a block. No term falls with batch, n_slots, kappa or capacity.
inline Layout layout(const PlanInputs* m, int batch, int n_slots, int kappa, int capacity) {
  const msd_model_config& c = m->cfg;
  const int64_t M = (int64_t)batch * n_slots;
  const int kmax = kappa > 1 ? kappa : 1;
  const int qd = c.n_heads * c.head_dim;
  Layout L{};
  L.MT = row_tiles(M);
  const RowPlan& rows = m->rows[L.MT - 1];
  L.s = rows.s;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += align_up(bytes);
    return o;
  };
  L.x = take((size_t)M * c.d_model * sizeof(float));
  L.stats = take((size_t)(c.d_model / kTileN) * M * sizeof(float2));
  // q as the attention's operand image: per sequence and kv head, the GQA
  // group's queries in 16-row tiles, hi + lo bf16 parts
  const int64_t q_tiles = ((int64_t)(c.n_heads / c.n_kv_heads) * n_slots + 15) / 16;
  L.q = take((size_t)batch * c.n_kv_heads * q_tiles * (c.head_dim / 32) * 1024 * sizeof(uint16_t));
  L.img_x = take(img_bytes(c.d_model, L.MT));
  L.img_h = take(img_bytes(c.d_model, L.MT));
  L.img_f = take(img_bytes(c.d_model, L.MT));
  L.img_attn = take(img_bytes(qd, L.MT));
  L.img_act = take(img_bytes(c.d_ffn, L.MT));
  // the GEMMs' split-K counters, then the attention's chunk counters (one per
  // sequence, kv head and query tile); all cleared by the rows kernel
  L.n_gemm_counters = rows.split_tiles;
  L.n_counters = rows.split_tiles + (int64_t)batch * c.n_kv_heads * q_tiles;
  L.counters = take((size_t)L.n_counters * sizeof(int32_t));
  L.max_chunks = (capacity + kAttnChunk - 1) / kAttnChunk;
  const size_t qn = (size_t)(c.n_heads / c.n_kv_heads) * n_slots;
  const size_t nparts = (size_t)batch * c.n_kv_heads * L.max_chunks * qn;
  // the GEMMs' and the attention's partials share one region: a GEMM's are read
  // by its own last kernel, the attention's by its own, and every kernel of a
  // step runs after the one before it
  const size_t shared = off;
  L.part_o = take(nparts * c.head_dim * sizeof(float));
  L.part_ml = take(nparts * sizeof(float2));
  const size_t attn_end = off;
  off = shared;
  L.partial = take(rows.part_bytes);
  off = std::max(off, attn_end);
  L.split_bytes = off - attn_end + align_up((size_t)L.n_counters * sizeof(int32_t)) -
                  align_up((size_t)(L.n_counters - L.n_gemm_counters) * sizeof(int32_t));
  L.tile_ms = take((size_t)rows.head_tiles * M * sizeof(float2));
  L.tile_top = take((size_t)rows.head_tiles * M * kmax * sizeof(uint64_t));
  const int parts = head_parts(rows.head_tiles);
  L.head_ms = take((size_t)parts * M * sizeof(float2));
  L.head_top = take((size_t)parts * M * kmax * sizeof(uint64_t));
  L.total = off;
  return L;
}

// Whether the static scratch holds a block: its workspace without the split
// partials and counters within MSD_STATIC_SCRATCH_BYTES.
inline bool fits_static(const Layout& L) {
  return L.total <= kStaticScratchBytes && L.total - L.split_bytes <= MSD_STATIC_SCRATCH_BYTES;
}

}  // namespace msd
