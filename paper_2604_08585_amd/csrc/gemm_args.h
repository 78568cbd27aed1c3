// Arguments of the bf16 product kernels, and their division by rows.  Plain host code as well (no HIP header).
#pragma once

#include <stdint.h>

struct qcf_chunk;

namespace qcf {

typedef uint16_t bf16_t;   // raw bfloat16 bits

// Re-rotation of the chunk caches (qcf_rerope) by workgroups behind those of the product, on the compute units that it leaves idle.
// Rows that the product writes (its dst_rows) are left out.
struct SideRerope {
  const qcf_chunk* chunks;
  int64_t total_rows;
  int n_chunks, style;
  int first_wg;                  // workgroups from here on (none: beyond the grid)
  int rows;                      // of each of them
};
constexpr int kSideRows = 192, kSideChunks = 256;      // rows worked on at a time; chunks, at most

struct QkvArgs {
  const bf16_t* x;
  const bf16_t* w;
  const int32_t* gather;
  const int32_t* pos;            // [M] absolute positions (rotary embedding; unused by the plain linear map)
  double neg2_over_d_log2base;   // theta_i = 2^(i * this)
  int64_t x_rows, M;
  int d_model, H, Hkv, D;
  int m_tiles, n_tiles;          // row tiles and 128-column blocks of this launch
  int n_tile0;                   // first block of this launch
  int m_group;                   // row tiles walked together (workgroup order of the 256 x 256 kernel)
  int rows_over_xcds;            // workgroup order of the load/compute-split kernel (see there)
  int splits, split_len;         // the contraction is cut into `splits` ranges of split_len k-tiles
  void* part;                    // their partial sums (splits > 1), float4
  bf16_t* q;
  bf16_t* k;
  bf16_t* v;
  // plain linear map (qcf_linear): all H*D columns go to q without rotation, or with the residual added (kAdd)
  const bf16_t* residual;
  // gated SiLU: block b holds weight rows 64 b .. +63 (gate) and glu + 64 b .. +63 (up) and gives
  // 64 output columns
  int glu;
  // projection fused with the write-back: row m of the K and V tiles also goes to row dst_rows[m] of the fused
  // cache (rows outside [0, fused_rows) are skipped); all null / 0 otherwise
  const int32_t* dst_rows;
  bf16_t* k_fused;
  bf16_t* v_fused;
  int64_t fused_rows;
  SideRerope side;
};

// What the epilogue does with a block: rotary embedding (half-split pairs of 128- or 64-wide heads, interleaved
// pairs), nothing, a residual, or the gated SiLU.  A template parameter: with all of them behind branches in one
// kernel the compiler moves accumulators of the k-loop to scratch.
enum Epi { kRopeHalf128, kRopeHalf64, kRopeInter, kPlain, kAdd, kGlu };
constexpr bool is_rope(int epi) { return epi <= kRopeInter; }

// The arguments of the same product without its first `rows` rows (a multiple of 256, so alignments stay).  An output that is
// NULL, i.e. not wanted, stays NULL: the kernels skip a block by that alone.
template <int EPI>
inline QkvArgs rows_from(QkvArgs a, int64_t rows) {
  const int64_t q_cols = EPI == kGlu ? a.glu : (int64_t)a.H * a.D, kv_cols = (int64_t)a.Hkv * a.D;
  if (a.gather) a.gather += rows;
  else { a.x += rows * a.d_model; a.x_rows -= rows; }
  if (a.pos) a.pos += rows;
  if (a.dst_rows) a.dst_rows += rows;
  if (a.q) a.q += rows * q_cols;
  if (a.residual) a.residual += rows * q_cols;
  if (a.k) a.k += rows * kv_cols;
  if (a.v) a.v += rows * kv_cols;
  a.M -= rows;
  return a;
}

}  // namespace qcf
