// Attention over the patched cache: arguments and device helpers shared by its kernels.
#pragma once

#include <type_traits>

#include "qcf_internal.h"

namespace qcf {
namespace attn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef short shortx8 __attribute__((ext_vector_type(8)));

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ int find_request(const int64_t* __restrict__ off, int B, int64_t row) {
  int b = 0;
  while (b < B && row >= off[b + 1]) ++b;
  return b;
}

struct AttnArgs {
  const void* q;
  const void* k;
  const void* v;
  const int32_t* sel_pos;
  const int64_t* sel_off;
  const int64_t* ctx_off;
  const int32_t* ctx_pos0;
  int64_t total_sel, total_ctx;
  int B, H, Hkv, G, D;
  int block_rows;        // selected rows of a row block (MFMA path)
  void* o;
  float* lse;
  int n_row_blocks;      // upper bound on row blocks over all requests (MFMA path)
  int seg_tiles;         // key tiles per work unit; a row block with more tiles is split over units
  int n_seg_max;         // units per row block the grid provides
  void* part_o;          // [unit][rows of a workgroup][D] normalised partial outputs of split row blocks (AttnTile<D>::part_t; float for the wide workgroups)
  float* part_lse;       // [unit][rows of a workgroup] log2-domain log-sum-exp of each partial (-inf: no visible key); d = 64: pairs of
                         // reference point (log2 units) and denominator against it
  int32_t* units;        // units[0] = number of work units, then (row block << 8 | segment), longest first (null: no plan)
  int32_t* blk_tiles;    // [row block] key tiles of the block, written by the plan kernel for the merge kernel (null: no plan)
};

constexpr int kBKV = 64;                    // tokens per K/V tile
template <int D>
struct AttnTile {
  static constexpr int ROW = 2 * D;                     // bytes of a staged row, no padding (swizzled instead)
  static constexpr int TILE = kBKV * ROW;               // bytes of a key or value tile
  static constexpr int STAGE = 2 * TILE;
  static constexpr size_t LDS = 2 * STAGE;
  static constexpr int LROWS = 1024 / ROW;              // rows filled by one load instruction of a wave (1 KB)
  static constexpr int NLOAD = kBKV / (4 * LROWS);      // instructions per wave and tile
  static constexpr int KS = D / 16, DT = D / 32;        // k-steps of the logits, 32-element slices of the output
  static constexpr int WG_ROWS = 128;                   // (selected row, head-in-group) pairs per workgroup
  static constexpr int WGS = 2;                         // resident workgroups per compute unit (registers)
  static constexpr bool SPLIT_P = D == 64;              // probabilities as three bf16 terms, fp32 partial outputs,
                                                        // rows that are not finite computed again
  typedef typename std::conditional<SPLIT_P, float, bf16_t>::type part_t;
  static constexpr float K2 = kLog2e * (D == 128 ? 0.08838834764831845f : 0.125f);      // log2(e) / sqrt(D)
};
// Slot of 16-byte chunk c of token row r inside the row, keys and values (see the layouts below).
template <int D> __device__ __forceinline__ int k_slot(int c, int r) { return D == 128 ? c ^ (r & 15) : c ^ ((r >> 1) & 7); }
template <int D> __device__ __forceinline__ int v_slot(int c, int r) { return D == 128 ? c ^ (4 * (r & 3)) : c ^ (4 * ((r >> 1) & 1)); }
constexpr float kLazyRescale = 8.f;         // log2 units the running maximum may lag behind the true one

// LDS transposing read: within each group of 16 lanes, lane i receives element i%4 of the four
// 8-byte rows addressed by lanes i/4, 4 + i/4, 8 + i/4, 12 + i/4 of the group.
__device__ __forceinline__ shortx4 lds_read_tr(uint32_t lds_addr) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)(uintptr_t)lds_addr);
}
// 16-byte LDS read at a byte address (a register plus a compile-time constant becomes the offset field)
__device__ __forceinline__ u32x4 lds_read16(uint32_t lds_addr) {
  return *(const u32x4 __attribute__((address_space(3)))*)(uintptr_t)lds_addr;
}

// Log-sum-exp of logits whose maximum is m / kLog2e and whose sum against it is 2^lz.  EXACT (heads of 64, and the wide workgroups): rounded once,
// and with the reciprocal of the kLog2e that m was scaled by (as two floats), not with ln 2.
template <bool EXACT>
__device__ __forceinline__ float natural_lse(float m, float lz) {
  if (!EXACT) return (m + lz) * kLn2;
  if (m == -INFINITY) return m;
  constexpr float lo = (float)(1.0 / (double)kLog2e - (double)kLn2);
  return __builtin_fmaf(m, kLn2, __builtin_fmaf(m, lo, lz * kLn2));
}
// Main kernel for heads of 128 with 256 rows to a workgroup, one workgroup to a compute unit (attn128.hip).
constexpr int kWideRows = 256;
qcf_status run_attn128(const AttnArgs& a, int64_t n_wg, hipStream_t st);

}  // namespace attn
}  // namespace qcf
