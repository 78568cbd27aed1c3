// How the attention of the MFMA kernels is divided into workgroups.  Plain host code as well (no HIP header).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "qcf.h"

namespace qcf {

int compute_unit_count();

namespace attn {

constexpr int kBKV = 64;                    // tokens per K/V tile
constexpr int kNarrowRows = 128, kWideRows = 256;      // (selected row, head-in-group) pairs of a workgroup
constexpr int kPlanMaxBlocks = 4096;        // row blocks a split launch may have (LDS table of the plan kernel)

// Key tiles per work unit.  With enough row blocks the causal triangle balances by itself and blocks
// stay whole; otherwise a segment is about the average causal work of a resident workgroup.
inline int resident_workgroups(int rows) { return (rows == kWideRows ? 1 : 2) * compute_unit_count(); }
constexpr int kShortTiles = 8, kShortSegments = 12;
struct Split { int seg_tiles, n_seg_max; bool part_f32 = false; };      // part_f32: partial outputs of heads of 128 in float
inline Split choose_split(int rows, int64_t n_blocks, int64_t total_ctx) {
  const int slots = resident_workgroups(rows);
  const int64_t n_t = std::max<int64_t>(1, (total_ctx + kBKV - 1) / kBKV);
  const int64_t per_slot = n_blocks * ((n_t + 1) / 2) / slots;     // average causal work per resident workgroup
  // a little above that average (a multiple of 4 tiles): most resident workgroups then take one whole
  // segment and the remainders fill the rest (measured best at recompute ratios 0.05, 0.15 and 0.30)
  int64_t seg = std::max<int64_t>(kShortTiles, (per_slot * 27 / 25 + 3) / 4 * 4);
  while ((n_t + seg - 1) / seg > 256) seg *= 2;       // a unit's segment number is kept in 8 bits
  if (n_blocks > kPlanMaxBlocks) seg = n_t;            // (never the case when splitting pays: see per_slot)
  if (seg >= n_t) return Split{(int)std::min<int64_t>(n_t, 0x3fffffff), 1};
  return Split{(int)seg, (int)((n_t + seg - 1) / seg)};
}

// Short launches of one request, which choose_split would give segments of kShortTiles tiles or none: a unit that has a compute
// unit to itself (half of the block-segment pairs lie above the diagonal and end at once) takes 1.26 us per tile, so shorter
// segments pay until their partial outputs, the merge's loop over them and its launch weigh more.  Their partial outputs are
// float: rows that were not divided before are not rounded once more.  Estimate in microseconds behind what every launch takes.
// Attention calls, us, as choose_split has it and so, 32 query and 8 KV heads of 128: 77 rows over 512 tokens 14.4 and 13.8,
// 96 over 640 18.9, 15.0; 30 over 731 19.3, 13.5; 110 over 731 19.0, 16.0; 150 over 1000 19.3, 17.4; 60 over 1500 19.5, 16.5;
// 100 over 2048 20.2, 20.1.  The other side of the line: 40 rows over 448 13.2 whole and in segments of 2; 225 over 1500 20.9 in
// segments of 8, 21.7 of 6; 307 over 2048 25.8, 27.9; 120 over 3000 22.2, 24.4.  Heads of 64: 110 over 731 20.9, 14.9; 100 over
// 2048 22.3, 18.9; 307 over 2048 28.8, 27.2; with 16 segments, 60 over 6000, 25.8 and 28.8.
inline Split short_split(int head_dim, double filled_blocks, int64_t total_ctx, Split general) {
  const int64_t n_t = std::max<int64_t>(1, (total_ctx + kBKV - 1) / kBKV);
  const bool whole = general.n_seg_max == 1;
  if (whole ? n_t > 2 * kShortTiles : general.seg_tiles > kShortTiles) return general;
  auto segments = [&](int64_t s) { return (int)((n_t + s - 1) / s); };
  auto units = [&](int64_t s) { return filled_blocks * ((double)n_t / (2.0 * (double)s) + 0.5); };
  auto us = [&](int64_t s, double per_unit) { return 1.26 * (double)s + per_unit * units(s) + 0.3 * segments(s) + 4.2; };
  double best = whole ? 1.26 * (double)n_t : us(kShortTiles, head_dim == 128 ? 0.02 : 0.03);
  Split sp = general;
  for (int64_t s = 2; s <= kShortTiles && s < n_t; ++s) {
    if (units(s) > compute_unit_count() || segments(s) > kShortSegments) continue;
    const double t = us(s, head_dim == 128 ? 0.035 : 0.03) + 0.3;
    if (t < best) { best = t; sp = Split{(int)s, segments(s), true}; }
  }
  return sp;
}

// How a launch is divided: rows of a workgroup, row blocks of all requests (upper bound), key segments.
struct Division { int rows; int64_t n_row_blocks; Split split; };
inline int64_t row_blocks(const qcf_layer_desc& L, int rows, int32_t B, int64_t total_sel) {
  const int br = rows / (L.n_q_heads / L.n_kv_heads);
  return (total_sel + br - 1) / br + B;
}
// 128 or 256 rows to a workgroup (heads of 128).  The wide workgroups read every key and value fragment half as often, but
// one of them fills a compute unit, so nothing hides the start and the end of its unit, a unit is the grain of the balance,
// and their partial outputs are fp32.  They take over where a compute unit's average causal work is long enough and the rows
// fill their blocks (0.92 of them, counted with one more than there are).  Narrow and wide, us, one request, 32 / 8 heads:
// 1228 rows over 12288 tokens (58 tiles to a compute unit) 142 and 150, 819 over 16384 (51) 139 and 140; 1843 over 12288
// (87) 202 and 190, 2457 over 8192 (77) 192 and 187, 2457 over 16384 (154) 358 and 339; 64 / 8 heads, 4915 over 32768 2468
// and 2262.  Blocks not filled: 64 / 8 heads, 491 rows over 24576 (0.90) 223 and 240; 32 / 32 heads, 876 over 23078 (0.68)
// 244 and 306, 2572 over 8509 (0.84) 215 and 227.  Of 256 launches of 50 to 420 tiles the best side of each would be 5.4 %
// faster than the narrow one everywhere, this rule 4.7 %, and one launch loses more than 1.5 % (4.5).
constexpr int64_t kWideTiles = 72;          // average causal work of a compute unit, in tiles (one request)
constexpr double kWideFill = 0.92;
// Several requests, of which the host knows the totals.  Narrow workgroups take 1.12 times as long for the same rows, but a
// request leaves a quarter of a 256-row block empty on average where its rows go in blocks of 128, half of one where they
// go in blocks of 256, and the start and end of a wide unit, which nothing hides, cost about seven of its tiles, those of
// a narrow one two.  With less than 512 tiles of work to a compute unit the last units decide, and the wide ones lose more
// often than not.  Narrow and wide, us, 32 query and 8 KV heads:
//   130 requests of 100 tokens, 5 rows each, 63 and 99; 128 of 512, 77 rows 208 and 296; 55 of 4096, 204 rows 575 and 828;
//   40 of 1500, 225 rows 203 and 240; 25 of 4096, 614 rows (244 tiles to a compute unit) 612 and 653 on one machine, 616 and
//   617 on another; 24 of 1K to 9K, 12 % of the rows (380) 1059 and 1095; 13 of 8192, 1228 rows (503) 1132 and 1250;
//   25 of 12288, 614 rows (723) 1860 and 1820; 12 of 1K to 12K, 26 % (720) 1727 and 1654; 17 of 12288, 1843 rows (1476)
//   3202 and 2954; 12 of 16384, 2457 rows (1850) 3855 and 3587.
// 272 batches of up to 256 requests: the worst that goes to the wide workgroups loses 2 %.
constexpr int64_t kWideBlocks = 4;          // row blocks to a compute unit
constexpr int64_t kWideBatchTiles = 512;    // average causal work of a compute unit
inline bool takes_wide(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx, int64_t blocks) {
  const double cus = compute_unit_count(), requests = (double)B * L.n_kv_heads;
  const double filled = (double)total_sel * L.n_q_heads / kWideRows;                 // row blocks without the empty rows
  const double tiles = ((double)total_ctx / B / kBKV + 1.0) / 2.0;                   // that a row sees, on average
  if (B == 1) return filled * tiles >= kWideTiles * cus && filled >= kWideFill * blocks;
  return blocks >= kWideBlocks * cus && filled * tiles >= kWideBatchTiles * cus &&
         1.12 * (filled + 0.25 * requests) * (tiles + 2.0) >= 1.01 * (filled + 0.5 * requests) * (tiles + 7.0);
}
inline Division divide_plainly(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx) {
  auto of = [&](int rows) {
    const int64_t nb = row_blocks(L, rows, B, total_sel);
    return Division{rows, nb, choose_split(rows, nb * L.n_kv_heads, total_ctx)};
  };
  if (L.head_dim == 128) {
    const Division wide = of(kWideRows);
    if (takes_wide(L, B, total_sel, total_ctx, wide.n_row_blocks * L.n_kv_heads)) return wide;
  }
  return of(kNarrowRows);
}

// Element of the partial outputs: float, but for the 128-row workgroups of heads of 128 in launches that are not short, which
// round them to bf16 (1229 rows x 32 heads over 8192 tokens write and read 20 MB of them so).
constexpr bool part_is_f32(int D, int rows, const Split& s) { return D == 64 || rows == kWideRows || s.part_f32; }

// What a split launch keeps in the workspace, in this order: partial outputs, their log-sum-exps (heads of 64: pairs), the list of
// units, the lengths of the row blocks.
inline size_t aligned(size_t n) { return (n + 255) / 256 * 256; }
inline size_t part_o_bytes(const qcf_layer_desc& L, const Division& d) {
  const size_t elem = part_is_f32(L.head_dim, d.rows, d.split) ? 4 : 2;
  return aligned((size_t)d.n_row_blocks * L.n_kv_heads * d.split.n_seg_max * d.rows * L.head_dim * elem);
}
inline size_t part_lse_bytes(const qcf_layer_desc& L, const Division& d) {
  return aligned((size_t)d.n_row_blocks * L.n_kv_heads * d.split.n_seg_max * d.rows * (L.head_dim == 128 ? 1 : 2) * sizeof(float));
}
inline size_t units_bytes(const Division& d) { return aligned((size_t)(d.n_row_blocks * d.split.n_seg_max + 1) * sizeof(int32_t)); }
inline size_t blk_tiles_bytes(const Division& d) { return aligned((size_t)d.n_row_blocks * sizeof(int32_t)); }
inline size_t workspace_of(const qcf_layer_desc& L, const Division& d) {
  if (d.split.n_seg_max <= 1) return 0;
  return part_o_bytes(L, d) + part_lse_bytes(L, d) + units_bytes(d) + blk_tiles_bytes(d);
}

// The division of a launch with ws_bytes of workspace.  Short segments keep more than choose_split's, and the more the fewer rows
// there are, so they are for a workspace that holds them: what a call has to be given (least_workspace) does not follow
// from them, and one workspace serves the layers of a model whatever the number of their rows.
inline Division divide(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx, size_t ws_bytes = SIZE_MAX) {
  const Division plain = divide_plainly(L, B, total_sel, total_ctx);
  if (B != 1 || plain.rows != kNarrowRows) return plain;
  Division d = plain;
  d.split = short_split(L.head_dim, (double)total_sel * L.n_q_heads / kNarrowRows, total_ctx, plain.split);
  return workspace_of(L, d) <= ws_bytes ? d : plain;
}
inline size_t least_workspace(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx) {
  return workspace_of(L, divide_plainly(L, B, total_sel, total_ctx));
}
inline size_t full_workspace(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx) {
  return std::max(least_workspace(L, B, total_sel, total_ctx), workspace_of(L, divide(L, B, total_sel, total_ctx)));
}

}  // namespace attn
}  // namespace qcf
