// Attention over the patched cache: arguments and device helpers shared by its kernels.
#pragma once

#include <type_traits>

#include "qcf_internal.h"
#include "attn_layout.h"

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
  void* part_o;          // [unit][32 rows][32 D] normalised partial outputs of split row blocks, in the order of the registers (attn_merge_kernel); float or bf16 (part_is_f32)
  float* part_lse;       // [unit][rows of a workgroup] log2-domain log-sum-exp of each partial (-inf: no visible key); d = 64: pairs of
                         // reference point (log2 units) and denominator against it
  int32_t* units;        // units[0] = number of work units, then (row block << 8 | segment), longest first (null: no plan)
  int seg_major;         // without a plan, > 0: row blocks whose segments of one number follow each other (one request: all with rows)
  int own_order;         // without a plan, 1: every workgroup finds its unit in that order itself (ordered_unit)
  int32_t* blk_tiles;    // [row block] key tiles of the block, written by the plan kernel for the merge kernel (null: no plan)
};

template <int D>
struct AttnTile {
  static constexpr int ROW = 2 * D;                     // bytes of a staged row, no padding (swizzled instead)
  static constexpr int TILE = kBKV * ROW;               // bytes of a key or value tile
  static constexpr int STAGE = 2 * TILE;
  static constexpr size_t LDS = 2 * STAGE;
  static constexpr int LROWS = 1024 / ROW;              // rows filled by one load instruction of a wave (1 KB)
  static constexpr int NLOAD = kBKV / (4 * LROWS);      // instructions per wave and tile
  static constexpr int KS = D / 16, DT = D / 32;        // k-steps of the logits, 32-element slices of the output
  static constexpr int WG_ROWS = kNarrowRows;           // (selected row, head-in-group) pairs per workgroup
  static constexpr int WGS = 2;                         // resident workgroups per compute unit (registers)
  static constexpr bool SPLIT_P = D == 64;              // probabilities as three bf16 terms, fp32 partial outputs,
                                                        // rows that are not finite computed again
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

// Log-sum-exp of logits whose maximum is m / kLog2e and whose sum against it is 2^lz.  EXACT (heads of 64, and the whole blocks
// of the wide workgroups; their split ones come from the merge, whose partials hold m + lz rounded once already): rounded
// once, and with the reciprocal of the kLog2e that m was scaled by (as two floats), not with ln 2.
template <bool EXACT>
__device__ __forceinline__ float natural_lse(float m, float lz) {
  if (!EXACT) return (m + lz) * kLn2;
  if (m == -INFINITY) return m;
  constexpr float lo = (float)(1.0 / (double)kLog2e - (double)kLn2);
  return __builtin_fmaf(m, kLn2, __builtin_fmaf(m, lo, lz * kLn2));
}
// Unit number `rank` of a split launch of one request, as (row block << 8 | segment), where the units are ordered by length
// (longest first) and from the last row block to the first among those of one length bucket.  Every workgroup of the launch
// works the same order out from the positions, which takes it about a microsecond (a launch that writes the order down takes
// five to six, in which nothing else runs).  A row block's length is taken from its last row; it bears on the order alone,
// so that rows in any order of positions are right.  All pairs that there may be have a place: those without tiles come last.
// `lds` is scratch of kOrderLds bytes, free again on return.
constexpr int kOrderMax = 512;              // units (row blocks x segments)
constexpr int kOrderBlocks = 256;           // row blocks, one to a thread
constexpr int kOrderBins = 64;              // lengths in 63rds of a segment: one to a lane
constexpr int kOrderLds = (kOrderBlocks + kOrderMax + kOrderBins) * 4;
__device__ __forceinline__ int ordered_unit(const AttnArgs& a, int rank, void* lds) {
  int* s_tiles = static_cast<int*>(lds);
  int* s_bin = s_tiles + kOrderBlocks;
  int* s_count = s_bin + kOrderMax;
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t s0 = min(max(a.sel_off[0], (int64_t)0), a.total_sel), s1 = min(max(a.sel_off[1], s0), a.total_sel);
  const int64_t c0 = min(max(a.ctx_off[0], (int64_t)0), a.total_ctx), c1 = min(max(a.ctx_off[1], c0), a.total_ctx);
  if (tid < a.n_row_blocks) {
    const int64_t first = s0 + (int64_t)tid * a.block_rows, last = min(first + a.block_rows, s1) - 1;
    int64_t vis = 0;
    if (last >= first) vis = min(c1 - c0, max((int64_t)0, (int64_t)a.sel_pos[last] - (a.ctx_pos0 ? a.ctx_pos0[0] : 0) + 1));
    s_tiles[tid] = (int)((vis + kBKV - 1) / kBKV);
  }
  if (tid < kOrderBins) s_count[tid] = 0;
  __syncthreads();
  const int n = a.n_row_blocks * a.n_seg_max;
  for (int u = tid; u < kOrderMax; u += 256) {
    int bin = -1;
    if (u < n) {
      const int len = s_tiles[a.n_row_blocks - 1 - u / a.n_seg_max] - u % a.n_seg_max * a.seg_tiles;
      bin = kOrderBins - 1 - (int)((float)min(max(len, 0), a.seg_tiles) * (float)(kOrderBins - 1) / (float)a.seg_tiles);
      bin = min(max(bin, 0), kOrderBins - 1);
      atomicAdd(&s_count[bin], 1);
    }
    s_bin[u] = bin;
  }
  __syncthreads();
  const int count = s_count[lane];
  int before = count;                                   // units of the buckets up to this lane's
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int t = __shfl_up(before, d, 64);
    if (lane >= d) before += t;
  }
  before -= count;
  const int bin = __popcll(__ballot(before <= rank)) - 1;      // the last bucket that starts at or before the rank: not an
  int left = rank - __shfl(before, bin, 64);                   // empty one, as rank < n
  int unit = 0;
#pragma unroll
  for (int i = 0; i < kOrderMax / 64; ++i) {
    const bool mine = s_bin[64 * i + lane] == bin;
    const uint64_t m = __ballot(mine);
    const uint64_t hit = __ballot(mine && (int)__popcll(m & ((1ull << lane) - 1)) == left);
    if (hit) unit = 64 * i + (int)__builtin_ctzll(hit);
    left -= (int)__popcll(m);
  }
  __syncthreads();
  unit = __builtin_amdgcn_readfirstlane(unit);
  return (a.n_row_blocks - 1 - unit / a.n_seg_max) << 8 | unit % a.n_seg_max;
}

// Main kernel for heads of 128 with kWideRows rows to a workgroup, one workgroup to a compute unit (attn128.hip).
qcf_status run_attn128(const AttnArgs& a, int64_t n_wg, hipStream_t st);

}  // namespace attn
}  // namespace qcf
