// How the products of the MFMA path are divided into launches and tiles, and which rows are re-rotated beside one.  Plain host
// code as well (no HIP header).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "gemm_args.h"
#include "qcf.h"

namespace qcf {

int compute_unit_count();

namespace gemm {

constexpr int kBK = 64;                  // contraction elements per LDS stage (rows of 128 bytes)
constexpr int kBN = 128;                 // columns of an output block: whole heads, or 64 gate + 64 up columns
constexpr int kQuadCols = 256;           // columns of a 256 x 256 tile

inline bool use_mfma(const qcf_layer_desc& L) {
  return L.dtype == QCF_DTYPE_BF16 && L.d_model % kBK == 0 && (L.n_kv_heads * L.head_dim) % kBN == 0;
}

// ---- choice of the tile --------------------------------------------------------------------------
// One workgroup per compute unit, so a launch takes (rounds of workgroups) x (time of one workgroup); the costs per
// k-tile and per workgroup are measured ones (microseconds, all compute units busy).  A split contraction adds the
// writing and reading of its partial sums and a launch.
enum GemmKind { kWs64, kWs96, kWs128, kWs160, kWs192, kWs224, kWs256, kQuad };       // 64 to 256 x 128; 256 x 256
constexpr int kRowsOf[] = {64, 96, 128, 160, 192, 224, 256, 256};
constexpr int rows_of(GemmKind kind) { return kRowsOf[kind]; }
struct GemmPlan { GemmKind kind; int splits; double us; };

inline double rounds_of(int64_t wgs) {
  const int cus = compute_unit_count();
  return (double)((wgs + cus - 1) / cus);
}
// Workgroups of a launch of mt row tiles with `units` (column blocks x ranges) to each: eight times those of the XCD that has most.
// (Column blocks are dealt to the XCDs with all their row tiles, or from kRowsOverXcds row tiles on the row tiles are; the numbers
// that are made up to a multiple of eight return at once.)
constexpr int64_t kRowsOverXcds = 16;
inline int64_t ws_grid(int64_t mt, int64_t units) {
  return mt >= kRowsOverXcds ? ((mt + 7) / 8) * 8 * units : mt * ((units + 7) / 8) * 8;
}
inline double quad_us(int64_t mt, int nb, int nk) { return rounds_of(mt * ((nb + 1) / 2)) * (1.40 * nk + 12.0); }
inline double ws256_us(int64_t mt, int nb, int nk) { return rounds_of(mt * nb) * (0.75 * nk + 10.0); }
// 128 x 128 tiles over three and more rounds wait for their operands: 2400 rows, K 8192, N 10240 take 0.7 us per k-tile.
// (With 0.45 there they were chosen: that layer took 1262 us, with two rounds of 256 x 256 tiles 1037.)
inline double ws128_tile_us(double rounds) { return rounds > 2 ? 0.65 : 0.45; }
inline double ws128_us(int64_t mt, int nb, int nk) {
  const double r = rounds_of(mt * nb);
  return r * (ws128_tile_us(r) * nk + 8.0);
}

// Tiles of other heights, where they fit one round.  These kernels are bound by their loads: a compute unit has at most 256 lines of
// 128 bytes on their way (60 GB/s from memory, 115 from the memory-side cache, whatever the depth of the ring), so a k-tile takes
// the time that its rows and columns take to arrive, and the least height that still fits a round wins.  Calls without and with
// them, us, of y = x w^T, weights from memory (buffers of 700 MB take turns): 64 rows: K 4096, N 6144 of 300 rows 35.8 and 30.6,
// K 2048, N 3072 of 615 21.0 and 17.8, K 2816, N 1024 of 2000 29.0 and 22.4, K 1024, N 1024 of 200 and 2000 8.7 and 8.4, 12.9 and
// 11.1; 96: K 4096, N 6144 of 350 34.9 and 32.0; 160: K 4096, N 4096 of 1229 52.5 and 45.9, K 2048, N 3072 of 1600 30.6 and 26.4;
// 192: K 4096, N 6144 of 900 54.3 and 49.3; 224: the same of 1100 58.0 and 55.4, K 8192, N 10240 of 615 110 and 106.  (Weights in
// the memory-side cache: 300 rows 24.5 and 23.4, 900 46.1 and 46.4, 1100 52.3 and 51.6.)  In two rounds they lose: K 4096,
// N 6144 of 410 rows in tiles of 64 54.0, of 96 32.5, of 128 35.7; 1229 in tiles of 160 85.8, of 256 58.4.
// A round is one of each XCD: where column blocks or row tiles are no multiple of eight, some have more workgroups than others.
// 560 rows of K 4096, N 3584 in 9 x 28 tiles of 64 (36 for 32 compute units) 49.4 us, in tiles of 96 33.6, of 128 31.7; 400 rows of
// N 4608 46.5, 28.9 and 30.2; 1865 of N 3200 in tiles of 192 82.4, of 256 54.8; 2305 of N 1152 in tiles of 96 48.1, of 128 37.6.
// Only up to K 8192: at K 14336 ranges of 256 x 256 tiles are faster than this says (N 4096 of 1290 rows 155 in ranges, 160 in tiles
// of 192; 1650 169 and 182).  (In between some would gain, K 11008, N 4096 of 1290 rows 148 and 126.)
struct Height { GemmKind kind; double tile_us, start_us; };
constexpr Height kHeights[] = {{kWs64, 0.44, 6.0}, {kWs96, 0.445, 6.0}, {kWs160, 0.61, 8.6}, {kWs192, 0.65, 8.5}, {kWs224, 0.72, 11.0}};
constexpr int kHeightTiles = 128;        // k-tiles, at most

// Tiles of 64 and 96 rows against 128 that fit a round too.  A last row tile with few rows runs ahead (the rows that it does not have
// are one line, which hits) and has the weights fetched for the others, so a k-tile takes, us, f the share of the last tile that has
// rows: 0.43 + 0.125 f of 128 rows, 0.40 + 0.10 f of 96, 0.375 + 0.0875 f of 64 (K 2048 and 4096, N 3072 to 6144 of 300 to 1000
// rows, within 4 %).  us, 128 and 96 rows: K 4096, N 4096 of 560 31.9 and 34.0, of 615 36.8 and 31.2; K 2048, N 3072 of 900 17.8 and 18.2,
// of 700 18.7 and 17.1; K 2816, N 1024 of 2200 23.2 and 25.6, of 2458 23.5 and 25.0; K 6144, N 2048 of 1400 57.9 and 49.2.
// One of 64 is before one of 96 where both pay, K 2816, N 1024 of 2000 rows 21.7 and 25.5, K 1536, N 2048 of 900 13.4 and 15.1, but not for
// contractions of up to kShortTiles k-tiles: K 256, N 512 of 1000 5.54 and 5.30 (128 rows 5.31), N 6144 of 160 5.58 and 5.48, K 512,
// N 2048 of 1000 7.27 and 6.82, K 1024, N 6144 of 300 11.4 and 10.8, N 1024 of 1229 9.11 and 8.92 (300: 8.53 and 8.59).
constexpr int kShortTiles = 18;
inline double last_tile_share(int64_t M, int rows) { return (double)((M - 1) % rows + 1) / rows; }
inline bool height_pays(GemmKind kind, int64_t M, int nk) {
  const double f = last_tile_share(M, rows_of(kind)), of128 = 0.43 + 0.125 * last_tile_share(M, 128);
  return kind == kWs96 ? 0.40 + 0.10 * f < of128 : kind == kWs64 && nk > kShortTiles && 0.375 + 0.0875 * f < of128;
}

// 256 x 256 tiles with the contraction in `s` ranges of an even number of k-tiles.  The partial sums leave all at once and
// are read again by the reduction (7 TB/s both ways: a hundred megabytes stay in the memory-side cache).  Few row tiles
// wait for their weights instead of the matrix unit; of two rounds the second's products hide the first's stores.
// Taken from 128 k-tiles on, over two rounds in three ranges or more (two would give a compute unit what the undivided tile
// gives it) of at least 64.  Product calls without and with it, us: K 14336, N 4096 of
// 400 rows 78 and 64, 768 rows 132 and 90, 1229 rows 178 and 130, 2458 rows 278 and 251; K 14336, N 9088 of 400 rows 181
// and 119; K 8192, N 10240 of 129 rows 69 and 55, 512 rows 111 and 89.  The other side of the line: K 4096, N 4096 of 1229
// rows 44 and 56, N 6144 of 700 rows 52 and 53 (a range of 22 k-tiles does not pay for its sums); K 8192, N 10240 of 900
// rows, two rounds of ranges of 44, 159 and 162; K 14336, N 4096 of 3300 rows, two rounds of two ranges, 303 and 338.
// (The 2.5 us behind the start are the launch of the reduction and its wait.  With 4.0, what it was when a workgroup of it finished 128
// columns by one wave, us so and with 2.5: K 14336, N 4096 of 300 rows 77.5 and 64.8, 1650 rows 186 and 169, K 8192, N 10240 of 390
// rows 86.1 and 84.5, all in tiles of 128 to 256 rows instead.)
// (Weights from memory.  In the memory-side cache, which has room for those of one product at best, the undivided tiles wait less:
// K 14336, N 4096 of 512 rows 61 and 65 there, 79 and 66 from memory, 1229 rows 145 and 125, 174 and 127; K 8192, N 10240 of
// 256 rows 51 and 60, 82 and 61.)
inline int quad_split_len(int nk, int s) { return (nk / 2 + s - 1) / s * 2; }
inline bool quad_split_pays(int64_t mt, int nb, int nk, int s) {
  const double r = rounds_of(mt * ((nb + 1) / 2) * s);
  return nk >= 128 && (r <= 1 || (r <= 2 && s >= 3 && quad_split_len(nk, s) >= 64));
}
inline double quad_split_us(int64_t mt, int nb, int nk, int s) {
  const double r = rounds_of(mt * ((nb + 1) / 2) * s);
  const double t = std::max(r * 1.36 * quad_split_len(nk, s), (double)nb * nk * (kBN * kBK * 2) / 4.6e6) + r * 6.0 + 2.5 +
                   (double)mt * nb * (256 * kBN * 8) * s / 7.0e6;
  return r > 1 ? 0.92 * t : t;
}

inline size_t split_part_bytes(int64_t M, int nb, int bm, int splits) {
  return splits <= 1 ? 0 : (size_t)splits * nb * ((M + bm - 1) / bm) * bm * kBN * sizeof(float);
}

// Main launch of a contraction in `s` ranges of `len` k-tiles over one row tile, which streams its weights: a workgroup waits
// for memory (0.44 and 0.55 us per k-tile of 64 and 128 rows), all together for its bandwidth (the more compute units load,
// the more there is; ranges that start 4 KB, 32 k-tiles, apart get a fifth less), and the reduction takes a quarter of a
// microsecond per range beside what the partial sums take.  Calls in ranges, us, 61 rows: K 14336, N 4096 in 4, 6, 7, 8 and
// 12 of them 37.2, 31.1, 34.8, 29.0, 36.5; K 8192, N 8192 in 2, 3, 4 42.2, 34.1, 40.7; K 2048, N 2048 in 4 and 8 10.1, 11.2.
// 110 rows: 44.1, 37.3, 38.9, 37.2, 41.7; 49.6, 39.9, 43.3; K 4096, N 6144 in 3, 4, 5 21.5, 19.7, 21.9.  (With 4.6 TB/s for
// any launch, behind its start, the first of each three to five were chosen, and 8 of K 2048.)
// The weights come from memory, as they do where the layers of a model follow each other.  Repeated calls find those of
// one layer in the memory-side cache (256 MB), where fewer ranges are a little better: 110 rows of K 4096, N 6144 in 3 and 4
// ranges 24.0 and 22.2 us from memory, 19.2 and 20.0 from the cache; the layer of 731 tokens with that projection 73.8 and
// 72.0 where twelve layers take turns, 64.2 and 64.8 where one is repeated.
inline double stream_us(int bm, int nb, int nk, int s, int len) {
  const double r = rounds_of((int64_t)nb * s), share = std::min(1.0, (double)nb * s / compute_unit_count());
  const double tb_s = (3.6 + 1.5 * share) * (s > 1 && len % 32 == 0 ? 0.82 : 1.0);
  return std::max(r * (bm == 64 ? 0.44 : 0.55) * len + r * 6.0, (double)nb * nk * (kBN * kBK * 2) / (tb_s * 1e6)) +
         (s > 1 ? 0.25 * s : 0.0);
}

// the load/compute-split kernels, over nb column blocks, with at most part_bytes of partial sums; `heights`: in tiles of any
// height (not where the cache is re-rotated beside the product, on the compute units that larger tiles leave idle).  They stand in
// for undivided tiles only, so that a product has one order of sums with the cache re-rotated beside it and without.  In place of
// ranges they lose as well: K 1536, N 2048 of 100 rows 12.1 us in ranges and 14.4 in tiles of 64 (15.3 of 96), 200 rows 13.5 and 13.6;
// K 2816, N 1024 of 1300 rows 22.6 and 22.2 (26.5); K 4096, N 12288 of 100 rows 34.5 and 34.9.
inline GemmPlan plan_ws(int64_t M, int nb, int nk, size_t part_bytes, bool heights) {
  GemmPlan best{kWs256, 1, ws256_us((M + 255) / 256, nb, nk)};
  const double t128 = ws128_us((M + 127) / 128, nb, nk);
  if (t128 < best.us) best = GemmPlan{kWs128, 1, t128};
  const int bm = M <= 64 ? 64 : 128;
  const int64_t tiles = (M + bm - 1) / bm * nb;
  const double c = bm == 64 ? 0.40 : ws128_tile_us(rounds_of(tiles));
  for (int s = 1; s <= 16 && s * 4 <= nk; ++s) {
    if (split_part_bytes(M, nb, bm, s) > part_bytes || (s > 1 && nb > 65535)) break;      // (grid.y of the reduction)
    const int len = (nk + s - 1) / s;
    if ((nk + len - 1) / len != s) continue;                     // (a range would be empty)
    double t = tiles == nb ? stream_us(bm, nb, nk, s, len)
                           : std::max(rounds_of(tiles * s) * c * len, (double)nb * nk * (kBN * kBK * 2) / 4.6e6) + rounds_of(tiles * s) * 6.0;
    if (s > 1) t += 4.0 + (double)tiles * bm * kBN * 8.0 * s / 4.0e6;
    if (t < best.us) best = GemmPlan{bm == 64 ? kWs64 : kWs128, s, t};
  }
  if (heights && best.splits == 1 && M > 64 && nk <= kHeightTiles) {
    auto fits = [&](GemmKind kind) { return ws_grid((M + rows_of(kind) - 1) / rows_of(kind), nb) <= compute_unit_count(); };
    const bool over128 = best.kind == kWs128 && fits(kWs128);
    for (const Height& h : kHeights) {
      const double t = h.tile_us * nk + h.start_us;
      if (!fits(h.kind) || !(over128 ? best.kind == kWs128 && height_pays(h.kind, M, nk) : t < best.us)) continue;
      best = GemmPlan{h.kind, 1, t};
    }
  }
  return best;
}

// The whole product: up to two launches.  The first, in tiles of `kind`, covers `rows` rows of all blocks or `blocks`
// blocks of all rows (rows == M and blocks == nb: everything, and only then in several ranges, `splits`); `rest` is the rest.
//
// A tile fills whole rounds of compute units only, so where the last round would be thin the first launch takes what
// full rounds hold and smaller tiles the rest: the column blocks that are left (256 x 256 tiles), or the rows that are
// left (tiles of 256 rows), whose contraction may be split because they are few.  Without the division by rows and with
// it, both sides in turn: K 4096, N 6144 of 1281 .. 1408 rows 75.2 .. 76.8 and 71.3 .. 74.5 us (its nearest edge; weights
// not in any cache: 77.0 and 74.2 .. 77.1), 2561 rows 126.8 and 115.2, 5377 rows 227.3 and 218.8; K 8192, N 10240 of 769
// rows 139.3 and 130.8, 4916 rows 627 and 594; K 14336, N 4096 of 2100 rows 235 and 205.  Where the rest is too long to
// be split the estimates are less good: 1500 and 2100 rows of the first shape lose 2.7 and 3.7 us.
// (128 x 128 tiles for the whole rounds lose: tail of 1229 rows 483 us in one launch, 492 that way.)
struct ProductPlan { GemmKind kind; int64_t rows; int blocks; GemmPlan rest; double us; int splits = 1; };

// The 256 x 256 kernel takes k-tiles in pairs, and its lanes address 256 weight rows with 32-bit byte offsets.
inline bool quad_ok(int nk) { return nk % 2 == 0 && (uint64_t)nk * kBK * 2 * kQuadCols <= (1ull << 32); }

inline ProductPlan plan_product(int64_t M, int nb, int nk, bool by_rows, size_t part_bytes, bool heights = true) {
  const GemmPlan one = plan_ws(M, nb, nk, part_bytes, heights);
  ProductPlan best{one.kind, 0, 0, one, one.us};                 // (rows and blocks 0: `rest` is everything)
  const int cus = compute_unit_count();
  const int64_t mt = (M + 255) / 256;
  if (quad_ok(nk)) {
    const double whole = quad_us(mt, nb, nk);
    if (whole < best.us) best = ProductPlan{kQuad, M, nb, one, whole};
    for (int s = 2; s <= 8 && nb <= 65535; ++s) {                // (grid.y of the reduction)
      if (split_part_bytes(M, nb, 256, s) > part_bytes) break;
      const int len = quad_split_len(nk, s);
      if ((nk + len - 1) / len != s || !quad_split_pays(mt, nb, nk, s)) continue;      // (a range would be empty)
      const double t = quad_split_us(mt, nb, nk, s);
      if (t < best.us) best = ProductPlan{kQuad, M, nb, one, t, s};
    }
    const int64_t rounds = mt * ((nb + 1) / 2) / cus;
    for (int64_t r = rounds; r >= 1 && r >= rounds - 1; --r) {
      const int qb = (int)(r * cus / mt * 2);
      if (qb <= 0 || qb >= nb) continue;
      // (`rest` in tiles of 128 or 256 rows, here and below: the estimates of two launches do not tell where others win.  K 4096, N
      // 6144 of 3250 rows 157 us, with tiles of 160 148; of 3000 141, with 96 146; N 28672 of 600 143 and 144.)
      const GemmPlan rest = plan_ws(M, nb - qb, nk, 0, false);
      const double t = quad_us(mt, qb, nk) + rest.us + 2.0;
      if (t < best.us) best = ProductPlan{kQuad, M, qb, rest, t};
    }
  }
  if (!by_rows) return best;
  for (GemmKind kind : {kQuad, kWs256}) {
    if (kind == kQuad && !quad_ok(nk)) continue;
    const int64_t units = kind == kQuad ? (nb + 1) / 2 : nb;     // workgroups of a row tile
    const int64_t rounds = mt * units / cus;
    for (int64_t r = rounds; r >= 1 && r >= rounds - 1; --r) {
      const int64_t tiles = r * cus / units;
      if (tiles <= 0 || tiles >= mt) continue;
      const GemmPlan rest = plan_ws(M - tiles * 256, nb, nk, part_bytes, false);
      const double t = (kind == kQuad ? quad_us(tiles, nb, nk) : ws256_us(tiles, nb, nk)) + rest.us + 2.0;
      // (256 x 256 tiles that fill half a round run faster than estimated, 256 x 128 tiles over several rounds slower:
      // 4200 rows, K 4096, N 6144 lost 28 us where 3 us were promised, 1500 rows 7 us where 14 were)
      if (t < best.us * (kind == kQuad ? 1.0 : 0.85)) best = ProductPlan{kind, tiles * 256, nb, rest, t};
    }
  }
  return best;
}

// workspace a product of M rows x nb column blocks x nk k-tiles can use (not needed: without it the contraction stays whole)
inline size_t gemm_part_bytes(int64_t M, int nb, int nk) {
  const ProductPlan p = plan_product(M, nb, nk, true, SIZE_MAX);
  if (p.blocks == nb && p.rows == M) return split_part_bytes(M, nb, 256, p.splits);
  return split_part_bytes(p.blocks == nb ? M - p.rows : M, p.blocks > 0 && p.blocks < nb ? nb - p.blocks : nb,
                          p.rest.kind == kWs64 ? 64 : 128, p.rest.splits);
}

// Re-rotation beside the product: rows of the cache for each workgroup and for all of them, the first ones (0: none; those behind
// them come from a launch in front).  It goes beside one launch of tiles of 64 to 256 rows that leaves compute units idle: all
// rows, if those are done with them before a launch of its own and the product would be one after the other, or as many as
// they get done meanwhile.  Layers of 8B shape that are not scored, us, with the launch and without: 110 rows over 731 tokens 43.9
// and 35.3, 410 over 4096 73.6, 66.1; 410 over 8192 93.4, 83.5; 480 over 12000 120.6, 111.9; 900 over 3000 (tiles of 256 rows)
// 105.0, 96.2; with a part of the rows (16 compute units idle) 615 over 4096 85.2, 83.3; 1229 over 8192 179.6, 176.6.
struct SideRows { int64_t each, all; };
inline SideRows side_rows(const qcf_layer_desc& L, int64_t M, int32_t n_chunks, int64_t total_rows, size_t ws_bytes) {
  const SideRows none{0, 0};
  if (!use_mfma(L) || M <= 0 || n_chunks > kSideChunks || (uint64_t)total_rows * L.d_model * 2u >= (1ull << 32)) return none;
  const int nb = (L.n_q_heads + 2 * L.n_kv_heads) * L.head_dim / kBN;
  const ProductPlan p = plan_product(M, nb, L.d_model / kBK, true, ws_bytes, false);
  if (p.blocks != 0) return none;
  const int bm = rows_of(p.rest.kind);
  const int64_t idle = compute_unit_count() - ws_grid((M + bm - 1) / bm, (int64_t)nb * p.rest.splits);
  if (idle < 8) return none;
  const double row_us = L.n_kv_heads * L.head_dim * 8e-6 / 44e-3, start = 5.0;      // 44 GB/s read and written by a compute unit
  const double alone = 2.0 + (double)total_rows * row_us / 125.0;                   // (5.5 TB/s by all of them)
  const int64_t each = (total_rows + idle - 1) / idle;
  if ((double)((each + kSideRows - 1) / kSideRows) * start + (double)each * row_us <= p.us + alone) return {each, total_rows};
  const int64_t fit = (int64_t)((0.9 * p.us - start) / (row_us + start / kSideRows));
  if (fit <= 0 || (double)(fit * idle) * row_us / 125.0 < 2.0) return none;
  return {fit, fit * idle};
}

}  // namespace gemm
}  // namespace qcf
