// Which scoring kernels a call takes, and how each of them divides its workspace.  The sizes that the library reports and
// the ones that its launches use come from the same functions.  Plain host code as well (no HIP header).
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "qcf.h"

namespace qcf {

int compute_unit_count();

namespace scoring {

constexpr int kTokPerWg = 256;                  // tokens of a tile
constexpr int kRowBlock = 320;                  // probe rows (of one group) staged in LDS at a time
constexpr int kMaxLayers = 16;                  // layers scored by one set of launches
constexpr int kSyncWords = 1024;                // counters of a single-kernel launch: finished workgroups, groups, tiles
constexpr size_t kPair = 2 * sizeof(float);     // a row's partial: (maximum, sum)

inline size_t aligned(size_t n) { return (n + 255) / 256 * 256; }

// upper bound on the 256-token tiles of all requests (tiles start at request boundaries: every request adds at
// most one partly filled tile); exact for a single request
inline int64_t n_tiles_upper(int32_t B, int64_t total_ctx) { return (total_ctx + (int64_t)B * (kTokPerWg - 1)) / kTokPerWg; }

inline bool use_mfma(const qcf_layer_desc& L) { return L.dtype == QCF_DTYPE_BF16 && (L.head_dim == 128 || L.head_dim == 64); }
inline size_t generic_ws(const qcf_layer_desc& L, int64_t total_probe, int64_t total_ctx) {
  return aligned((size_t)total_probe * L.n_q_heads * total_ctx * sizeof(float));
}

// Two passes: the partials of every unit of tiles, then the column sums.
struct PassWs { int unit_tiles; int64_t n_units; size_t colsum, total; };
inline PassWs pass_ws_of(const qcf_layer_desc& L, int n_layers, int unit_tiles, int64_t n_units, int64_t total_probe,
                         int64_t total_ctx) {
  PassWs w;
  w.unit_tiles = unit_tiles;
  w.n_units = n_units;
  w.colsum = aligned((size_t)n_layers * n_units * total_probe * L.n_q_heads * kPair);
  w.total = w.colsum + aligned((size_t)n_layers * L.n_kv_heads * total_ctx * sizeof(float));
  return w;
}
// Units of all requests, upper bound.  A request of nt tiles has ceil(nt / unit_tiles) units: every request may end in a unit
// that is not full, but none has more units than tiles (with more requests than tokens the first bound is the larger).
inline int64_t n_units_upper(int32_t B, int64_t total_ctx, int unit_tiles) {
  const int64_t nt = n_tiles_upper(B, total_ctx);
  return std::min(nt, (nt + (int64_t)B * (unit_tiles - 1)) / unit_tiles);
}
// Tiles that a workgroup of the two passes takes in turn.  A workgroup spends about as long on staging probe rows and on its
// sums as on kUnitCost tiles; where a launch is a few rounds long whole rounds count, otherwise the tail is about half a
// unit.  (32768 tokens, 8 KV heads: units of four tiles, one round; with one tile to a unit pass 2 alone took 149 us, now 71.)
// Of several requests the host knows the totals.  The estimate takes their lengths to be uneven, which counts up to a tile too
// many for each; requests of one length that fit one round of the chip by that reading are asked for first:
//   - one tile to a unit fits, and the bound adds no more than a quarter of a round of workgroups without a tile, or the rows
//     take several blocks, for each of which a larger unit stages its keys again.  4 requests of 4000 tokens x 16 heads of 64:
//     16 probe rows 17.1 us, with two tiles to a unit 21.2; 160 rows 39 and 57.  16 of 500 x 64 heads of 128: 160 rows 86 and
//     118, but 16 rows 37 and 32;
//   - with well over one block of rows, the smallest unit that fits: 16 of 1000, 160 rows x 64 heads of 128, one tile (two
//     rounds) 148, two 136, four 193; 16 of 2000 285, 245 and 213.
constexpr double kUnitCost = 1.5;
inline int unit_tiles_for(int32_t B, int64_t total_probe, int64_t total_ctx, int64_t heads_layers, int64_t group) {
  const int64_t nt = n_tiles_upper(B, total_ctx);
  const double cus = compute_unit_count();
  int best = 1;
  double best_cost = 0;
  for (int ul = 1; ul <= 64 && ul <= nt; ++ul) {
    const double per_cu = (double)((nt + ul - 1) / ul + (B - 1) / 2) * (double)heads_layers / cus;
    const double cost = (per_cu <= 3.0 ? ceil(per_cu) : per_cu + 0.5) * (ul + kUnitCost);
    if (ul == 1 || cost < best_cost) { best = ul; best_cost = cost; }
  }
  if (B == 1) return best;
  const int64_t tiles = std::max<int64_t>(1, (total_ctx + (int64_t)kTokPerWg * B - 1) / ((int64_t)kTokPerWg * B));
  const double rows = (double)total_probe * group / B;
  auto fits = [&](int64_t units) { return (double)units * heads_layers <= cus; };
  if (fits(B * tiles)) return (double)nt * heads_layers <= 1.25 * cus || rows > kRowBlock ? 1 : best;
  if (rows > 1.5 * kRowBlock)
    for (int ul = 2; ul < best; ++ul)
      if (fits(B * ((tiles + ul - 1) / ul))) return ul;
  return best;
}
// What the launches of n_layers layers use.
inline PassWs pass_ws(const qcf_layer_desc& L, int n_layers, int32_t B, int64_t total_probe, int64_t total_ctx) {
  const int unit_tiles = unit_tiles_for(B, total_probe, total_ctx, (int64_t)L.n_kv_heads * n_layers, L.n_q_heads / L.n_kv_heads);
  return pass_ws_of(L, n_layers, unit_tiles, n_units_upper(B, total_ctx, unit_tiles), total_probe, total_ctx);
}
// The size reported for one layer: one tile to a unit, at least what pass_ws gives.
inline size_t two_pass_bytes(const qcf_layer_desc& L, int32_t B, int64_t total_probe, int64_t total_ctx) {
  return pass_ws_of(L, 1, 1, n_tiles_upper(B, total_ctx), total_probe, total_ctx).total;
}
// Heads of 64 keep the generic kernels where many short requests would make the partials (one per started 256 tokens)
// larger than its probability rows and than the built-in scratch of qcf_score_static.
inline bool use_two_pass(const qcf_layer_desc& L, int32_t B, int64_t total_probe, int64_t total_ctx) {
  return use_mfma(L) && (L.head_dim == 128 || two_pass_bytes(L, B, total_probe, total_ctx) <=
                             std::max(generic_ws(L, total_probe, total_ctx), (size_t)QCF_SCORE_STATIC_SCRATCH_BYTES));
}

// The single-kernel path needs every workgroup of the launch resident at once (one per compute unit) and all
// probe rows of a KV group in one staged block.  The host only knows totals, so the test is on those.  Heads of 64 never
// take it: their calls may overlap on any number of streams, which the counter sets of this path (kSyncSlots) and its wait
// for workgroups that another launch may keep off the chip do not allow.
inline bool use_fused(const qcf_layer_desc& L, int32_t B, int64_t total_probe, int64_t total_ctx) {
  if (!use_mfma(L) || L.head_dim != 128 || total_probe <= 0) return false;
  const int64_t G = L.n_q_heads / L.n_kv_heads;
  const int64_t tiles = n_tiles_upper(B, total_ctx);
  return total_probe * G <= kRowBlock && tiles * L.n_kv_heads <= compute_unit_count() &&
         1 + (int64_t)B * L.n_kv_heads + tiles <= kSyncWords;
}
// Re-rotation in the same launch (no probe_limit): one request whose chunk table the kernel keeps in LDS, and no more than two fillings
// of its (cos, sin) pairs to a tile on average.  Critical layers of 8B shape, us, re-rotation as a launch and so: 731 tokens
// in 16 chunks (5.6 to a tile) 57.2 and 55.0, 45 (15.8) 57.4 and 57.8, 128 (45) 57.3 and 60.9; 300 in 16 (13.7) 52.9 and 51.6, 30 (26)
// 53.4 and 54.6; 2000 in 128 (16.4) 68.3 and 66.6.
constexpr int kMaxRotChunks = 128, kRotChunksPerTile = 16;
inline bool takes_rerope(const qcf_layer_desc& L, int32_t B, int32_t n_chunks, int64_t total_probe, int64_t total_ctx) {
  return B == 1 && n_chunks > 0 && n_chunks <= kMaxRotChunks && n_chunks * (int64_t)kTokPerWg <= kRotChunksPerTile * total_ctx + kTokPerWg &&
         use_fused(L, B, total_probe, total_ctx);
}
// what the kernel of pass 1 that re-rotates is made for
inline bool pass1_rerotates(const qcf_layer_desc& L, int unit_tiles, int n_layers, bool limit) {
  return L.head_dim == 64 && unit_tiles == 1 && n_layers == 1 && L.n_kv_heads <= 65535 && !limit;
}
// Re-rotation inside pass 1: heads of 64, one request in units of one tile that all start at once, chunks as above.  Layers
// of 32 / 8 heads, us, re-rotation as a launch and so: 8000 tokens (250 units) 178.7 and 177.1, 90 38.3 and 35.9, 4160 in 64 chunks
// 90.7 and 88.2, 900 in 60 (17 to a tile) 53.3 and 52.4.  Beyond the line nothing is gained: 12000 tokens (376 units) 321.7 and
// 321.0, 960 in 120 chunks (32 to a tile) 52.9 both ways.
inline bool pass1_takes_rerope(const qcf_layer_desc& L, int32_t B, int32_t n_chunks, int64_t total_probe, int64_t total_ctx) {
  return B == 1 && n_chunks > 0 && n_chunks <= kMaxRotChunks && total_probe > 0 && total_ctx > 0 &&
         n_chunks * (int64_t)kTokPerWg <= kRotChunksPerTile * total_ctx + kTokPerWg && use_mfma(L) &&
         use_two_pass(L, B, total_probe, total_ctx) && n_tiles_upper(B, total_ctx) * L.n_kv_heads <= compute_unit_count() &&
         pass1_rerotates(L, pass_ws(L, 1, B, total_probe, total_ctx).unit_tiles, 1, false);
}
struct FusedWs { size_t part, colpart, total; };
inline FusedWs fused_ws(const qcf_layer_desc& L, int32_t B, int64_t total_ctx) {
  const size_t slots = (size_t)n_tiles_upper(B, total_ctx) * L.n_kv_heads;
  FusedWs w;
  w.part = 0;
  w.colpart = aligned(slots * kRowBlock * kPair);
  w.total = w.colpart + aligned(slots * kTokPerWg * sizeof(float));
  return w;
}

// One layer.
inline size_t workspace(const qcf_layer_desc& L, int32_t B, int64_t total_probe, int64_t total_ctx) {
  if (use_fused(L, B, total_probe, total_ctx)) return fused_ws(L, B, total_ctx).total;
  if (use_two_pass(L, B, total_probe, total_ctx)) return two_pass_bytes(L, B, total_probe, total_ctx);
  return generic_ws(L, total_probe, total_ctx);
}
// Where a scoring call is followed by the selection over the same tokens, the selection's workgroup adds up the last sums itself: the
// KV heads' column sums of the two passes, or the generic path's probability rows.  One request, and no more to read than one
// compute unit gets through in about the time of the launch that it saves (some 100 KB a microsecond): 192 KB, of the generic
// path up to 512 tokens, where a token's rows are shared by two threads at least, and beyond 128 tokens up to the 96 rows that are on
// their way at once.  Whole layers, us, with the launch and without, in a captured graph: heads of 64 (8 KV heads), 40 probe rows
// over 256 tokens 45.7 and 42.8, 1024 55.4 and 52.7, 4096 (128 KB) 96.1 and 93.2; heads of 128, 100 over 300 64.5 and 61.1; f32, 4 heads,
// 20 rows over 64 23.2 and 21.9, 96 over 128 (192 KB) 27.8 and 27.4, 24 over 200 26.0 and 25.5.  The other side of the line: heads of
// 64, 6000 tokens (192 KB, and eight tokens to a thread) 139.9 and 149.4, 8192 201.3 and 212.8; f32, 8 heads, 20 rows over 300 (160 rows)
// 32.0 and 34.9, 4 heads, 36 over 180 (144) 26.1 and 26.6; 20 over 600 34.6 and 37.5.  Just inside it, f32 of 300 to 512 tokens and 80 to 96
// rows, a graph is slower (4 heads, 20 over 512 28.9 and 30.1), calls that the host enqueues take the same (31.5 and 31.5).
enum SumsOf { kNoSums, kHeads, kRows };
constexpr int kSumTokens = 4096, kSumRowTokens = 512;
constexpr int kSumFewTokens = 128, kSumRows = 96;
constexpr size_t kSumBytes = (size_t)192 << 10;
inline SumsOf sums_in_selection(const qcf_layer_desc& L, int32_t B, int64_t total_probe, int64_t total_ctx) {
  if (B != 1 || total_probe <= 0 || total_ctx <= 0 || total_ctx > kSumTokens || use_fused(L, B, total_probe, total_ctx)) return kNoSums;
  if (use_two_pass(L, B, total_probe, total_ctx)) return (size_t)L.n_kv_heads * total_ctx * sizeof(float) <= kSumBytes ? kHeads : kNoSums;
  if (total_ctx > kSumRowTokens || (total_ctx > kSumFewTokens && total_probe * L.n_q_heads > kSumRows)) return kNoSums;
  return generic_ws(L, total_probe, total_ctx) <= kSumBytes ? kRows : kNoSums;
}

// Layers scored by one set of launches: as many as keep the workspace within that of a single call, or 64 MiB.  One where
// the two passes do not apply.
inline int layers_at_once(const qcf_layer_desc& L, int32_t n_layers, int32_t B, int64_t total_probe, int64_t total_ctx) {
  if (total_probe <= 0 || L.head_dim != 128 || !use_two_pass(L, B, total_probe, total_ctx)) return 1;
  const size_t limit = std::max(workspace(L, B, total_probe, total_ctx), (size_t)64 << 20);
  int n = std::min(n_layers, kMaxLayers);
  while (n > 1 && pass_ws(L, n, B, total_probe, total_ctx).total > limit) --n;
  return n;
}
inline size_t layers_workspace(const qcf_layer_desc& L, int32_t n_layers, int32_t B, int64_t total_probe, int64_t total_ctx) {
  const int n = layers_at_once(L, n_layers, B, total_probe, total_ctx);
  size_t need = workspace(L, B, total_probe, total_ctx);
  if (n > 1) need = std::max(need, pass_ws(L, n, B, total_probe, total_ctx).total);
  if (n > 1 && n_layers % n > 1) need = std::max(need, pass_ws(L, n_layers % n, B, total_probe, total_ctx).total);
  return need;
}

}  // namespace scoring
}  // namespace qcf
