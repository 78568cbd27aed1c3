// Step 2: critical-layer attention analysis (Section 3.1 Phase 3; Section 3.2 token
// selector of the paper): score[j] = mean over probe rows and heads of the softmax
// attention the context token j receives.
//
// bf16 / head_dim 128 and 64 path (the dense contraction runs on MFMA).  A workgroup of twelve waves takes a unit of
// 256-token tiles of one KV head: the group's probe rows arrive in LDS once per unit, the keys of one tile after the
// other, through asynchronous loads that request every 128-byte line once (loading keys straight into registers in MFMA
// operand layout touches 64 different lines per instruction, which is what bounded the earlier version);
// wave (tw, rg) keeps the 64 tokens of slice tw in registers and takes every third 32-row tile of the rows.  The keys of
// the next tile travel while the current one is used.
//   pass 1  logits of the probe rows against the tiles -> per-row (max, sum-exp) of the unit, in the log2
//           domain (the four token slices folded in LDS);
//   pass 2  every workgroup first folds the partials of its group's rows over the request's units into
//           a maximum and a sum per row (in a fixed order, so all workgroups get the same values); logits
//           again, p = exp2(logit - max) / sum, summed over the rows of the group -> per-KV-head column sums;
//   reduce  fixed-order sum over KV heads, times 1/(R*H), and over layers where several are scored at once.
// Bound by the exponentials and what goes with them (about 205 vector instructions, 1200 cycles of a SIMD, per 64 tokens x
// 32 rows and pass, against 512 of MFMAs) and, with few probe rows, by the keys: 8 layers, 48 rows x 32 heads over 6001
// tokens 170 us in eight launches of the single kernel below, 32 + 33 + 5 us here, where the loads alone take 21 + 22; 80
// rows x 64 heads over 32768 tokens 85 + 149 us with one tile to a workgroup, whose every workgroup of pass 2 folded 128
// partials per row, 60 + 61 here.  A wave's next MFMAs between the exponentials of its last rows (two waves to a SIMD, no
// registers for a third): 77 + 82.
// Launches that are resident at once (one workgroup per compute unit at most, up to 320 probe rows per KV
// group) take a single kernel instead (score_fused, further down): the exponentials of pass 1 stay in registers
// across a grid-wide exchange of the per-row partials, so the keys are read once and no second pass or reduce
// kernel runs.  For a layer of one request it turns the keys as well (RR).
// No floating-point atomics anywhere, so scores (and the indices selected from them) are
// bit-stable from run to run.
//
// Heads of 64 run the two MFMA passes with half the k-steps (40 probe rows x 32 heads over 4096 tokens: 391 us with the
// generic kernels, 15.7 us here), never the single kernel (see use_fused).
//
// Generic path (f32, or other head dims): one workgroup per (probe row, head) materialises its
// softmax row in the workspace, then a column mean.
#include <type_traits>

#include "qcf_internal.h"
#include "score_layout.h"

namespace qcf {
using namespace scoring;
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr float kLog2e = 1.4426950408889634f;

// request owning global row `row` given offsets[0..B]; returns B if none
__device__ __forceinline__ int find_request(const int64_t* __restrict__ off, int B, int64_t row) {
  int b = 0;
  while (b < B && row >= off[b + 1]) ++b;
  return b;
}

// ------------------------------------------------------------------ generic path

// D / 4 lanes take a token, so that a load brings whole key rows, and a wave has eight of its loads on their way.  Up to
// kKeptLogits tokens the row's logits and exponentials stay in LDS; through the workspace every step waits for the stores of
// the one before.  Both kernels of a call, us, with one thread to a token and the row in the workspace, and so: 20 rows x 8 heads of
// 64 over 512 tokens 12.8 and 10.1, over 2000 25.9 and 15.9; 80 rows x 8 heads of 128 over 1000 tokens 63.5 and 38.6.
// THREADS: 512, of which a row of few tokens leaves most idle; several requests of 512 tokens or less on average take 256 (the
// whole call, us, 512 and 256: 200 requests of 64 tokens, 20 rows x 4 heads of 64, 260 and 143, 50 of 100 32.5 and 23.4, 16
// of 512 17.4 and 16.3; the other side of the line: 8 of 1000 16.2 and 17.2, one of 512 7.7 and 8.6).
constexpr int kRowLoads = 8;
constexpr int kKeptLogits = 2048;
constexpr int kShortTokens = 512;

template <typename T, int D, int THREADS>
__global__ __launch_bounds__(THREADS) void score_rows_generic(
    const T* __restrict__ q, const int64_t* __restrict__ probe_off, int64_t /*total_probe*/,
    const T* __restrict__ k, const int64_t* __restrict__ ctx_off, int64_t total_ctx, int B,
    const int32_t* __restrict__ probe_limit, int H, int Hkv, float* __restrict__ P) {
  constexpr int kRowThreads = THREADS, kRowWaves = kRowThreads / 64;
  constexpr int kLanes = D / 4, kTokens = 64 / kLanes;           // lanes of a token, tokens of a load
  static_assert(D == 64 || D == 128, "a row of 16 lanes, or two");
  __shared__ float red[2][kRowWaves];
  __shared__ float kept[kKeptLogits];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = blockIdx.x / H;
  const int h = blockIdx.x - (int)row * H;
  float qf[4];
  Quad<T>::load(q + ((int64_t)row * H + h) * D + 4 * (lane % kLanes), qf);
  const int b = find_request(probe_off, B, row);
  if (b >= B) return;
  int64_t c0 = min(max(ctx_off[b], (int64_t)0), total_ctx);
  int64_t c1 = min(max(ctx_off[b + 1], c0), total_ctx);
  const int Tn = (int)(c1 - c0);
  int limit = Tn;
  if (probe_limit) limit = min(Tn, max(0, probe_limit[row]));
  float* prow = P + ((int64_t)row * H + h) * total_ctx + c0;
  const int g = h / (H / Hkv);
  const float scale = rsqrtf((float)D);
  auto softmax_row = [&](float* w) {
    const int step = kTokens * kRowLoads;
    for (int j0 = wave * step; j0 < limit; j0 += kRowWaves * step) {
      float kf[kRowLoads][4];
#pragma unroll
      for (int u = 0; u < kRowLoads; ++u) {
        const int j = min(j0 + u * kTokens + lane / kLanes, limit - 1);
        Quad<T>::load(k + ((c0 + j) * Hkv + g) * (int64_t)D + 4 * (lane % kLanes), kf[u]);
      }
#pragma unroll
      for (int u = 0; u < kRowLoads; ++u) {
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) acc += qf[e] * kf[u][e];
        acc = kLanes == 16 ? row_sum(acc) : half_wave_sum(acc);
        const int j = j0 + u * kTokens + lane / kLanes;
        if (lane % kLanes == 0 && j < limit) w[j] = acc * scale;
      }
    }
    __syncthreads();
    float mx = -INFINITY;
    for (int j = tid; j < limit; j += kRowThreads) mx = fmaxf(mx, w[j]);
    for (int d = 32; d >= 1; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
    if (lane == 0) red[0][wave] = mx;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kRowWaves; ++i) mx = fmaxf(mx, red[0][i]);
    float sum = 0.f;
    for (int j = tid; j < limit; j += kRowThreads) {
      const float e = expf(w[j] - mx);
      w[j] = e;
      sum += e;
    }
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) red[1][wave] = sum;
    __syncthreads();
    sum = 0.f;
#pragma unroll
    for (int i = 0; i < kRowWaves; ++i) sum += red[1][i];
    for (int j = tid; j < Tn; j += kRowThreads) prow[j] = (j < limit) ? w[j] / sum : 0.f;
  };
  if (limit <= kKeptLogits) softmax_row(kept);
  else softmax_row(prow);
}

// The columns of 64 tokens to a workgroup: every wave adds a contiguous share of the rows in order, kColRows of them on
// their way at a time, and the first one the waves' sums in order.  Both
// kernels of a call, us, with a thread to a token that adds all rows, and so: 20 rows x 8 heads over 512 tokens 10.1 and 8.5, 40 rows
// x 16 heads over 300 23.3 and 13.6, 80 rows x 8 heads of 128 over 1000 38.6 and 29.0.
constexpr int kColTokens = 64, kColWaves = 8, kColRows = 16;
__global__ __launch_bounds__(64 * kColWaves) void score_colmean_generic(
    const float* __restrict__ P, const int64_t* __restrict__ probe_off, int64_t total_probe,
    const int64_t* __restrict__ ctx_off, int64_t total_ctx, int B, int H, float* score, float alpha, float beta) {
  __shared__ float part[kColWaves][kColTokens];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t j = (int64_t)blockIdx.x * kColTokens + lane;
  const int b = j < total_ctx ? find_request(ctx_off, B, j) : B;
  int64_t r0 = 0, r1 = 0;
  if (b < B) {
    r0 = min(max(probe_off[b], (int64_t)0), total_probe);
    r1 = min(max(probe_off[b + 1], r0), total_probe);
  }
  const int64_t share = ((r1 - r0) * H + kColWaves - 1) / kColWaves;
  const int64_t end = min(r0 * H + (wave + 1) * share, r1 * H);
  float acc = 0.f;
  for (int64_t r = r0 * H + wave * share; r < end; r += kColRows) {
    float p[kColRows];
#pragma unroll
    for (int u = 0; u < kColRows; ++u) p[u] = P[min(r + u, end - 1) * total_ctx + j];
#pragma unroll
    for (int u = 0; u < kColRows; ++u) acc += r + u < end ? p[u] : 0.f;
  }
  part[wave][lane] = acc;
  __syncthreads();
  if (wave != 0 || b >= B) return;
  acc = 0.f;
#pragma unroll
  for (int w = 0; w < kColWaves; ++w) acc += part[w][lane];
  const float sj = (r1 > r0) ? acc / (float)((r1 - r0) * H) : 0.f;
  score[j] = (beta == 0.f) ? alpha * sj : __builtin_fmaf(beta, score[j], alpha * sj);
}

// ------------------------------------------------------------------ MFMA path (bf16, d = 128 or 64)

constexpr int kTokWaves = 4;                    // token slices of a workgroup
constexpr int kTokPerWave = kTokPerWg / kTokWaves;      // tokens a wave keeps stationary in registers
constexpr int kRowGroups = 3;                   // waves per token slice, which share a SIMD and share out the row tiles
constexpr int kWavesPerWg = kTokWaves * kRowGroups;
constexpr int kThreads = 64 * kWavesPerWg;
template <int D> constexpr size_t kQBytes = (size_t)kRowBlock * D * 2;     // staged rows: swizzled, no padding
template <int D> constexpr size_t kKBytes = (size_t)kTokPerWg * D * 2;
template <int D> constexpr float kK2 = kLog2e * (D == 128 ? 0.08838834764831845f : 0.125f);    // log2(e) / sqrt(D)
// Staged rows: a load instruction of a wave fills kRowsPerLoad rows (1 KB).  Chunk c (16 bytes) of row r sits in slot
// c ^ (r % 16) of its row (d = 128: a row is one sweep over the banks) or c ^ (r / 2 % 8) (d = 64: two rows are), so
// the 16-byte fragment reads of 16 consecutive rows touch 16 different bank groups.
template <int D> constexpr int kRowsPerLoad = 1024 / (2 * D);
template <int D> __device__ __forceinline__ int slot_of(int c, int r) { return D == 128 ? c ^ (r & 15) : c ^ ((r >> 1) & 7); }
// row, and the element offset of the chunk, that lane `lane` of staging instruction j brings
template <int D> __device__ __forceinline__ int staged_row(int j, int lane) { return kRowsPerLoad<D> * j + lane / (64 / kRowsPerLoad<D>); }
template <int D> __device__ __forceinline__ int staged_elem(int r, int lane) { return slot_of<D>(lane % (64 / kRowsPerLoad<D>), r) * 8; }
// byte offset of this lane's fragment (row lane%32, chunk 2*ks + lane/32) is frag_base ^ (32 * ks)
template <int D> __device__ __forceinline__ int frag_base(int lane) { return (lane & 31) * 2 * D + slot_of<D>(lane >> 5, lane & 31) * 16; }
constexpr int kFoldBatch = 16;
// The passes keep a row's maximum and the reciprocal of its sum apart instead of one log-sum-exp, whose rounding weighs
// once logits reach a hundred (heads of 64, largest logit 586: 8.7e-6 off in the 2-norm, now 1.7e-6, the general kernels
// 1.9e-6; largest 12: 1.6e-7, 8.3e-8, 5.3e-7; heads of 128, 80 rows over 32768 tokens: 1.9e-7, 7.0e-8).  Heads of 64: a NaN
// in either reaches every token that the row sees, the maximum is that of the unscaled logits and is taken off before they
// are scaled, so that the largest one gives exactly 1 at any magnitude.
template <int D> constexpr bool kPairs = D == 64;
template <int D> constexpr float kMaxScale = kPairs<D> ? kK2<D> : 1.f;      // from a kept maximum to log2 units
template <int D> __device__ __forceinline__ float exp_of(float logit, float m) {
  if (kPairs<D>) return __builtin_amdgcn_exp2f((logit - m) * kK2<D>);
  return __builtin_amdgcn_exp2f(__builtin_fmaf(logit, kK2<D>, -m));
}

struct ScoreArgs {
  const bf16_t* q;            // [total_probe, H, D]
  const bf16_t* k;            // [total_ctx, Hkv, D]
  const int64_t* probe_off;
  const int64_t* ctx_off;
  const int32_t* probe_limit;
  int64_t total_probe, total_ctx;
  int B, H, Hkv, G;
  float2* part;               // [layer][unit][total_probe * H] (max2, sumexp2) per unit of tiles
  float* colsum;              // [layer][Hkv][total_ctx]
  float* score;
  float alpha, beta;          // score = beta * score + alpha * (this call's mean attention); beta == 0: plain store
};

// plain store, or blended into what is there (accumulation over layers)
__device__ __forceinline__ float blended(float beta, float old, float s) { return (beta == 0.f) ? s : __builtin_fmaf(beta, old, s); }
__device__ __forceinline__ void write_score(const ScoreArgs& a, int64_t j, float s) {
  a.score[j] = blended(a.beta, (a.beta == 0.f) ? 0.f : a.score[j], a.alpha * s);
}

// Maps a workgroup index (= tile number over all requests) to (request, first token of its 256-token
// tile, number of the request's first tile).  Tiles are aligned to the start of each request.  Returns
// false when the index is past the last tile.
__device__ __forceinline__ bool locate_tile(const ScoreArgs& a, int wg, int& b, int64_t& c0, int& T,
                                            int& tile_tok0, int& tile_first) {
  tile_first = 0;
  for (b = 0; b < a.B; ++b) {
    c0 = min(max(a.ctx_off[b], (int64_t)0), a.total_ctx);
    const int64_t c1 = min(max(a.ctx_off[b + 1], c0), a.total_ctx);
    T = (int)(c1 - c0);
    const int nt = (T + kTokPerWg - 1) / kTokPerWg;
    if (wg < nt) {
      tile_tok0 = wg * kTokPerWg;
      return true;
    }
    wg -= nt;
    tile_first += nt;
  }
  return false;
}

// Brings the 256 key rows of a tile (tokens 256 * tile .. + 255 of KV head g) into LDS with asynchronous direct-to-LDS
// loads (1 KB per instruction, every 128-byte line requested once); same row layout as the probe rows below.  Tokens past
// the end of the request are clamped (masked or never written later).
template <int D>
struct KeyLoader {
  static constexpr int kLoads = kTokPerWg / kRowsPerLoad<D>;     // of the workgroup, per tile
  static constexpr int kStep = kRowsPerLoad<D> * kWavesPerWg;    // rows between those of a wave (the slots repeat)
  const char* base;                  // head g of the request's first token
  uint32_t row_bytes, row0, chunk, lds;
  int T;
  __device__ __forceinline__ KeyLoader(const bf16_t* head, int Hkv, int T_, uint32_t lds_k, int wave, int lane)
      : base(reinterpret_cast<const char*>(head)), row_bytes((uint32_t)Hkv * D * 2), row0((uint32_t)staged_row<D>(wave, lane)),
        chunk((uint32_t)staged_elem<D>((int)row0, lane) * 2), lds(lds_k + (uint32_t)wave * 1024), T(T_) {
    static_assert(kStep % 16 == 0, "rows kStep apart have the same slots");
  }
  __device__ __forceinline__ void load(int tile, int wave) const {
    const char* src = base + (int64_t)tile * kTokPerWg * row_bytes;
    const bool whole = tile * kTokPerWg + kTokPerWg <= T;
#pragma unroll
    for (int i = 0; i * kWavesPerWg < kLoads; ++i) {
      if ((i + 1) * kWavesPerWg > kLoads && i * kWavesPerWg + wave >= kLoads) break;
      const uint32_t row = row0 + (uint32_t)(kStep * i), dst = lds + (uint32_t)i * kWavesPerWg * 1024;
      if (whole) load_to_lds_at(src + (int64_t)(kStep * i) * row_bytes, row0 * row_bytes + chunk, dst);
      else load_to_lds_at(src, min(row, (uint32_t)(T - 1 - tile * kTokPerWg)) * row_bytes + chunk, dst);
    }
  }
};

// Key fragments of a wave's 64 tokens, from the first of their staged rows.
template <int D>
__device__ __forceinline__ void load_key_frags(const unsigned char* rows, int qb0, bf16x8 (&kf)[2][D / 16]) {
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
      kf[mt][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(rows + 32 * mt * (2 * D) + (qb0 ^ (32 * ks))));
}

// Logits of a wave's 64 tokens (key fragments kf) against the 32 staged probe rows at `rows` (LDS address of this lane's
// first fragment): the row fragments are requested up to four k-steps ahead of the MFMAs that use them.  TOKENS_FIRST: the
// result's rows are tokens (A = keys) and its columns probe rows (B = queries), else the other way round.
template <int D, bool TOKENS_FIRST>
__device__ __forceinline__ void logit_tile(const bf16x8 (&kf)[2][D / 16], uint32_t rows, floatx16& acc0, floatx16& acc1) {
  constexpr int KS = D / 16;
  auto read = [&](int ks) { return *(const u32x4 __attribute__((address_space(3)))*)(uintptr_t)(rows ^ (uint32_t)(32 * ks)); };
  u32x4 ring[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) ring[i] = read(i);
  acc0 = floatx16{0};
  acc1 = floatx16{0};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    __builtin_amdgcn_sched_barrier(0);
    const bf16x8 qf = __builtin_bit_cast(bf16x8, ring[ks & 3]);
    if (TOKENS_FIRST) {
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0][ks], qf, acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[1][ks], qf, acc1, 0, 0, 0);
    } else {
      acc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, kf[0][ks], acc0, 0, 0, 0);
      acc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf, kf[1][ks], acc1, 0, 0, 0);
    }
    if (ks + 4 < KS) ring[ks & 3] = read(ks + 4);
  }
}

// Stages probe rows [r_begin, r_begin + n_rows) of group g (row r = i*G + hh <-> probe row i,
// head g*G + hh) into LDS with asynchronous direct-to-LDS loads; the caller waits and synchronises.
// Rows up to the next multiple of 32 are filled with a copy of the last row (never used in a result).
template <int D>
__device__ __forceinline__ void stage_q_async(const ScoreArgs& a, const bf16_t* q, int64_t p0, int g, int r_begin, int n_rows,
                                              int n_rows_pad, uint32_t sQ, int wave, int lane) {
  for (int j = wave; j < n_rows_pad / kRowsPerLoad<D>; j += kWavesPerWg) {
    const int r = staged_row<D>(j, lane);
    const int rr = r_begin + min(r, n_rows - 1);
    const int i = rr / a.G, hh = rr - i * a.G;
    load_to_lds_addr_at(q + ((p0 + i) * a.H + g * a.G + hh) * D + staged_elem<D>(r, lane), sQ + j * 1024);
  }
}

// exchange between the two 32-lane halves of a wave (one vector instruction, no LDS round trip):
// returns the value the lane 32 away holds
__device__ __forceinline__ float other_half(float x) {
  typedef unsigned u2v __attribute__((ext_vector_type(2)));
  const u2v r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  // r.x = (lower half's value in both halves), r.y = (upper half's value in both halves)
  return (threadIdx.x & 32) ? __uint_as_float(r.x) : __uint_as_float(r.y);
}
// Both passes run over a set of layers at once (qcf_score_layers; one layer otherwise).  A workgroup takes the
// (up to unit_tiles) 256-token tiles of one unit of one request, for one KV head of one layer: the probe rows are
// staged once per unit, and the keys of the next tile travel while the current one, already in registers, is used.
struct PassArgs {
  ScoreArgs s;                       // (s.q, s.k and s.alpha belong to layer 0; the arrays below are used)
  const bf16_t* q[kMaxLayers];
  const bf16_t* k[kMaxLayers];
  float alpha[kMaxLayers];
  int n_layers;
  int unit_tiles;                    // most tiles of a unit
  uint32_t unit_magic;               // x * unit_magic >> 32 == x / unit_tiles, for x * unit_tiles < 2^32 and unit_tiles > 1
  int n_units;                       // units the grid provides (upper bound on the units of all requests)
};
struct Unit {
  int layer, g, b, T;
  int64_t c0;
  int tile0, tile1;                  // tiles of the request
  int64_t slot;                      // this unit's partials
  int64_t slot_first;                // partials of the request's first unit, and how many units it has
  int n_units;
};
// One layer in units of one tile, the short launches: the kernels come in a form of their own (ONE) that takes ScoreArgs, in a
// grid of (tile, head), keeps nothing from tile to tile and runs every row tile through the same code.  Such a launch
// waits for its arguments, its place and its instructions rather than for its arithmetic.  40 probe rows x 32 heads of 64 over
// 2048 tokens 17.7 us by the other form, 15.1 so; x 16 heads over 16384 23.0 and 19.1; 200 rows x 32 heads of 128 over 4096
// 49.5 and 43.8; 80 rows x 64 heads of 128 over 2048 38.6 and 34.7.
template <bool ONE> using Args = typename std::conditional<ONE, ScoreArgs, PassArgs>::type;
__host__ __device__ __forceinline__ const ScoreArgs& common(const ScoreArgs& a) { return a; }
__host__ __device__ __forceinline__ const ScoreArgs& common(const PassArgs& a) { return a.s; }
__device__ __forceinline__ const bf16_t* probes_of(const ScoreArgs& a, const Unit&) { return a.q; }
__device__ __forceinline__ const bf16_t* probes_of(const PassArgs& a, const Unit& u) { return a.q[u.layer]; }
__device__ __forceinline__ const bf16_t* keys_of(const ScoreArgs& a, const Unit&) { return a.k; }
__device__ __forceinline__ const bf16_t* keys_of(const PassArgs& a, const Unit& u) { return a.k[u.layer]; }
__device__ __forceinline__ bool locate_unit(const ScoreArgs& a, Unit& u) {
  int tok0, first;
  if (!locate_tile(a, (int)blockIdx.x, u.b, u.c0, u.T, tok0, first)) return false;
  u.layer = 0;
  u.g = (int)blockIdx.y;
  u.tile0 = tok0 / kTokPerWg;
  u.tile1 = u.tile0 + 1;
  u.slot = blockIdx.x;
  u.slot_first = first;
  u.n_units = (u.T + kTokPerWg - 1) / kTokPerWg;
  return true;
}
// The tiles of a request are dealt evenly to its units.  Consecutive workgroups take the KV heads in turn, so that with
// eight of them the units of a head, which read the same probe rows, share an XCD.
__device__ __forceinline__ bool locate_unit(const PassArgs& a, Unit& u) {
  const ScoreArgs& s = a.s;
  u.g = (int)(blockIdx.x % (unsigned)s.Hkv);
  const int rest = (int)(blockIdx.x / (unsigned)s.Hkv);
  u.layer = rest % a.n_layers;
  int idx = rest / a.n_layers, first = 0;
  for (u.b = 0; u.b < s.B; ++u.b) {
    u.c0 = min(max(s.ctx_off[u.b], (int64_t)0), s.total_ctx);
    const int64_t c1 = min(max(s.ctx_off[u.b + 1], u.c0), s.total_ctx);
    u.T = (int)(c1 - u.c0);
    const int nt = (u.T + kTokPerWg - 1) / kTokPerWg;
    // (a division for every request in front of the unit's: 64 requests of 300 tokens 158 us, 135 without)
    u.n_units = a.unit_tiles == 1 ? nt : (int)__umulhi((uint32_t)(nt + a.unit_tiles - 1), a.unit_magic);
    if (idx < u.n_units) {
      u.tile0 = (int)((int64_t)idx * nt / u.n_units);
      u.tile1 = (int)((int64_t)(idx + 1) * nt / u.n_units);
      u.slot_first = (int64_t)u.layer * a.n_units + first;
      u.slot = u.slot_first + idx;
      return true;
    }
    idx -= u.n_units;
    first += u.n_units;
  }
  return false;
}

constexpr int kTilesPerWave = (kRowBlock / 32 + kRowGroups - 1) / kRowGroups;      // row tiles of a wave, at most

// Re-rotation inside a scoring kernel (RR): the chunks whose keys and values make up the cache that s.k points to.
struct Rerotation {
  const qcf_chunk* chunks;
  int n_chunks, style;
  double neg2_over_d_log2base;
  bf16_t* k;                 // the fused cache, keys (s.k) and values
  bf16_t* v;
};

template <int D> constexpr size_t kPass1Lds = kQBytes<D> + kKBytes<D> + (size_t)kTokWaves * kRowBlock * sizeof(float2);
// Re-rotation of a unit's tile inside pass 1 (RR; heads of 64): the chunk table, each row's chunk and sources, and the pairs
// of the tile's chunks, behind pass 1's own LDS.
struct Pass1Rot {
  qcf_chunk table[kMaxRotChunks];
  const char* k[kTokPerWg];                       // source of a row, for this KV head (row of no chunk: itself)
  const char* v[kTokPerWg];
  int chunk[kTokPerWg];                           // last chunk that starts at or before a row
  bool covered[kTokPerWg];
  float2 cs[kMaxRotChunks * 32];
};
static_assert(sizeof(qcf_chunk) % 8 == 0, "copied in words of 8 bytes");
struct NoRerotation {};
template <bool RR> using RerotationOf = typename std::conditional<RR, Rerotation, NoRerotation>::type;

// One tile of one KV head by the whole workgroup: four threads to a row, two 16-byte vectors of keys (the partners of eight pairs) and of
// values each.  Keys are turned and left in LDS as load_key_frags wants them; store() then writes both to the cache, at the end of the
// kernel, where nothing waits for the stores.
struct TileRerotation {
  static constexpr int D = 64, kItems = (4 * kTokPerWg + kThreads - 1) / kThreads;
  u32x4 vals[kItems][2];
  int e0, de;                                     // first elements of a thread's two vectors
  // beside: loads of something else, requested behind the keys' and the values' (in front of them the barriers would wait for it)
  template <typename F>
  __device__ __forceinline__ void load(const Rerotation& r, Pass1Rot& rot, const ScoreArgs& a, const Unit& u, unsigned char* sK, F&& beside) {
    const int tid = threadIdx.x, n = min(kTokPerWg, u.T - u.tile0 * kTokPerWg);      // rows of the tile
    const int64_t row0 = u.c0 + (int64_t)u.tile0 * kTokPerWg, row_elems = (int64_t)a.Hkv * D;
    if (tid < n) {
      const int64_t row = row0 + tid;
      const int c = chunk_of(rot.table, r.n_chunks, row);
      const qcf_chunk& ch = rot.table[c];
      const bool covered = row >= ch.dst_row && row < ch.dst_row + ch.len;
      const int64_t off = ((covered ? row - ch.dst_row : row) * row_elems + u.g * D) * 2;
      rot.k[tid] = static_cast<const char*>(covered ? ch.k_src : r.k) + off;
      rot.v[tid] = static_cast<const char*>(covered ? ch.v_src : r.v) + off;
      rot.chunk[tid] = c;
      rot.covered[tid] = covered;
    }
    __syncthreads();
    const int p0 = 8 * (tid & 3);                 // (kThreads is a multiple of four: the same piece of every row)
    e0 = r.style == 0 ? p0 : 2 * p0;
    de = r.style == 0 ? D / 2 : 8;
    u32x4 keys[kItems][2];
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int row = (tid + i * kThreads) >> 2;
      if (row < n) {
        keys[i][0] = *reinterpret_cast<const u32x4*>(rot.k[row] + 2 * e0);
        keys[i][1] = *reinterpret_cast<const u32x4*>(rot.k[row] + 2 * (e0 + de));
        vals[i][0] = *reinterpret_cast<const u32x4*>(rot.v[row] + 2 * e0);
        vals[i][1] = *reinterpret_cast<const u32x4*>(rot.v[row] + 2 * (e0 + de));
      }
    }
    beside();
    const int first = rot.chunk[0], n_mine = rot.chunk[n - 1] - first + 1;
    for (int i = tid; i < n_mine * (D / 2); i += kThreads)
      rot.cs[i] = shift_pair(rot.table[first + i / (D / 2)], r.neg2_over_d_log2base, i % (D / 2));
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int row = (tid + i * kThreads) >> 2;
      if (row >= kTokPerWg) continue;
      if (row >= n) {                             // (masked tokens)
        keys[i][0] = mk4(0, 0, 0, 0);
        keys[i][1] = mk4(0, 0, 0, 0);
      } else if (rot.covered[row]) {
        const float2* cs = rot.cs + (rot.chunk[row] - first) * (D / 2) + p0;
        float f[16], o[16];
        Vec16<bf16_t>::unpack(keys[i][0], f);
        Vec16<bf16_t>::unpack(keys[i][1], f + 8);
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          float x, y;
          turn_pair(r.style == 0 ? f[p] : f[2 * p], r.style == 0 ? f[p + 8] : f[2 * p + 1], cs[p], x, y);
          if (r.style == 0) { o[p] = x; o[p + 8] = y; }
          else { o[2 * p] = x; o[2 * p + 1] = y; }
        }
        keys[i][0] = Vec16<bf16_t>::pack(o);
        keys[i][1] = Vec16<bf16_t>::pack(o + 8);
      }
      *reinterpret_cast<u32x4*>(sK + row * 2 * D + slot_of<D>(e0 / 8, row) * 16) = keys[i][0];
      *reinterpret_cast<u32x4*>(sK + row * 2 * D + slot_of<D>((e0 + de) / 8, row) * 16) = keys[i][1];
    }
  }
  __device__ __forceinline__ void store(const Rerotation& r, const Pass1Rot& rot, const ScoreArgs& a, const Unit& u, const unsigned char* sK) const {
    const int tid = threadIdx.x, n = min(kTokPerWg, u.T - u.tile0 * kTokPerWg);
    const int64_t row0 = u.c0 + (int64_t)u.tile0 * kTokPerWg, row_elems = (int64_t)a.Hkv * D;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const int row = (tid + i * kThreads) >> 2;
      if (row >= n || !rot.covered[row]) continue;
      const int64_t dst = (row0 + row) * row_elems + u.g * D + e0;
      *reinterpret_cast<u32x4*>(r.k + dst) = *reinterpret_cast<const u32x4*>(sK + row * 2 * D + slot_of<D>(e0 / 8, row) * 16);
      *reinterpret_cast<u32x4*>(r.k + dst + de) = *reinterpret_cast<const u32x4*>(sK + row * 2 * D + slot_of<D>((e0 + de) / 8, row) * 16);
      *reinterpret_cast<u32x4*>(r.v + dst) = vals[i][0];
      *reinterpret_cast<u32x4*>(r.v + dst + de) = vals[i][1];
    }
  }
};

// One row and KV head that no tile covers (cache rows outside the request), by one wave.
template <int D>
__device__ __forceinline__ void rerotate_row(const Rerotation& r, const qcf_chunk* table, int64_t row, int Hkv, int g, int lane) {
  const qcf_chunk ch = table[chunk_of(table, r.n_chunks, row)];
  if (row < ch.dst_row || row >= ch.dst_row + ch.len || lane >= D / 2) return;
  const int64_t src = (row - ch.dst_row) * Hkv * D + g * D, dst = row * Hkv * D + g * D;
  const bf16_t* k = static_cast<const bf16_t*>(ch.k_src) + src;
  const bf16_t* v = static_cast<const bf16_t*>(ch.v_src) + src;
  const int ia = r.style == 0 ? lane : 2 * lane, ib = r.style == 0 ? lane + D / 2 : 2 * lane + 1;
  float a, b;
  turn_pair(bf16_to_f32(k[ia]), bf16_to_f32(k[ib]), shift_pair(ch, r.neg2_over_d_log2base, lane), a, b);
  r.k[dst + ia] = f32_to_bf16(a);
  r.k[dst + ib] = f32_to_bf16(b);
  r.v[dst + lane] = v[lane];
  r.v[dst + D / 2 + lane] = v[D / 2 + lane];
}

// Pass 1.  Wave (tw, rg) keeps the 64 tokens of slice tw in registers and takes every third 32-row tile of the staged
// probe rows, starting with tile rg; a lane keeps the running (max, sum-exp) of its rows over the unit's tiles.
// RR (heads of 64, one request, one tile to a unit): the tile's keys come from the chunk caches, are turned on their way to LDS and
// written to the cache behind everything else, with the values.  Saves the launch of qcf_rerope and the reading of the keys; a chain
// of latencies, like score_fused's: 4096 tokens, 40 rows x 32 heads 6.6 + 6.8 us in two launches, 11.4 so (12.5 with the probe rows
// requested first, which the barriers in front of the keys' loads then wait for).  The layer 86.6 and 84.7 us, 90 tokens 38.3 and
// 35.9, 1230 53.8 and 52.4, 8000 178.7 and 177.1.
template <int D, bool LIMIT, bool ONE, bool RR>
__global__ __launch_bounds__(kThreads) void score_pass1(Args<ONE> pa, RerotationOf<RR> rr) {
  static_assert(!RR || (D == 64 && ONE && !LIMIT), "the form that re-rotates");
  const ScoreArgs& a = common(pa);
  extern __shared__ __align__(256) unsigned char smem[];      // (fragment addresses are formed with XORs below 256)
  unsigned char* sK = smem + kQBytes<D>;
  float2* sPart = reinterpret_cast<float2*>(smem + kQBytes<D> + kKBytes<D>);     // [kTokWaves][kRowBlock]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tw = wave % kTokWaves, rg = wave / kTokWaves;
  const uint32_t lds0 = lds_offset_of(smem);
  Unit u;
  Pass1Rot& rot = *reinterpret_cast<Pass1Rot*>(smem + kPass1Lds<D>);     // (RR)
  if constexpr (RR) {
    for (int i = tid; i < rr.n_chunks * (int)(sizeof(qcf_chunk) / 8); i += kThreads)
      reinterpret_cast<uint64_t*>(rot.table)[i] = reinterpret_cast<const uint64_t*>(rr.chunks)[i];
  }
  const bool have_unit = locate_unit(pa, u);
  if constexpr (RR) {
    __syncthreads();
    const int64_t lo = min(max(a.ctx_off[0], (int64_t)0), a.total_ctx), hi = min(max(a.ctx_off[1], lo), a.total_ctx);
    for (int64_t i = (int64_t)blockIdx.x * kWavesPerWg + wave; i < a.total_ctx - (hi - lo); i += (int64_t)gridDim.x * kWavesPerWg)
      rerotate_row<D>(rr, rot.table, i < lo ? i : i + (hi - lo), a.Hkv, (int)blockIdx.y, lane);
  }
  if (!have_unit) return;
  const int64_t p0 = min(max(a.probe_off[u.b], (int64_t)0), a.total_probe);
  const int64_t p1 = min(max(a.probe_off[u.b + 1], p0), a.total_probe);
  const int rows = (int)(p1 - p0) * a.G;         // probe rows x heads of the group
  TileRerotation turned;
  if constexpr (RR) {
    turned.load(rr, rot, a, u, sK, [&] {
      const int n = min(kRowBlock, rows);
      if (n > 0) stage_q_async<D>(a, probes_of(pa, u), p0, u.g, 0, n, (n + 31) & ~31, lds0, wave, lane);
    });
    if (rows == 0) {
      __syncthreads();
      turned.store(rr, rot, a, u, sK);
    }
  }
  if (rows == 0) return;
  const bf16_t* q = probes_of(pa, u);
  const KeyLoader<D> keys(keys_of(pa, u) + (u.c0 * a.Hkv + u.g) * D, a.Hkv, u.T, lds0 + (uint32_t)kQBytes<D>, wave, lane);
  const int qb0 = frag_base<D>(lane);
  float2* part = a.part + u.slot * (a.total_probe * a.H);

  for (int r_begin = 0; r_begin < rows; r_begin += kRowBlock) {
    const int n_rows = min(kRowBlock, rows - r_begin);
    const int n_pad = (n_rows + 31) & ~31;
    __syncthreads();                        // the previous block's rows and partials are no longer read
    if (ONE && !RR && r_begin == 0) keys.load(u.tile0, wave);      // (they stay in LDS)
    if (!RR || r_begin > 0) stage_q_async<D>(a, q, p0, u.g, r_begin, n_rows, n_pad, lds0, wave, lane);
    if (!ONE) keys.load(u.tile0, wave);
    // how many tokens the lane's row of row tile rt sees
    auto limit_of = [&](int rt) {
      const int r = r_begin + rt + (lane & 31);
      return LIMIT && r < r_begin + n_rows ? min(u.T, max(0, a.probe_limit[p0 + r / a.G])) : u.T;
    };
    // 64 tokens from tok0 on into a lane's running maximum (of the row) and sum (of this half of the tokens)
    auto add_tokens = [&](const bf16x8 (&kf)[2][D / 16], int rt, int tok0, int lim, float& m_run, float& z_run) {
      floatx16 acc0, acc1;
      logit_tile<D, true>(kf, lds0 + (uint32_t)(rt * 2 * D + qb0), acc0, acc1);
      // lane owns probe row rt + lane%32; its registers hold tokens 8*(v/4) + 4*(lane/32) + v%4
      float s[32];
#pragma unroll
      for (int v = 0; v < 16; ++v) { s[v] = acc0[v]; s[16 + v] = acc1[v]; }
      if (LIMIT || tok0 + kTokPerWave > u.T) {        // wave-uniform: only ragged or limited tiles compare
        const int left = lim - tok0 - 4 * (lane >> 5);
#pragma unroll
        for (int v = 0; v < 32; ++v) s[v] = (32 * (v >> 4) + 8 * ((v & 15) >> 2) + (v & 3) < left) ? s[v] : -INFINITY;
      }
      float mx = s[0];
#pragma unroll
      for (int v = 1; v < 32; ++v) mx = fmaxf(mx, s[v]);
      mx = fmaxf(mx, other_half(mx));
      if (!kPairs<D>) mx *= kK2<D>;                         // (positive: scaling commutes with the maximum)
      const float m_new = fmaxf(m_run, mx);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      float sum = z_run * __builtin_amdgcn_exp2f((m_run - m_use) * kMaxScale<D>);
#pragma unroll
      for (int v = 0; v < 32; ++v) sum += exp_of<D>(s[v], m_use);
      m_run = m_new;
      z_run = sum;
    };
    auto store = [&](int rt, float m, float z) {
      z += other_half(z);
      if (lane < 32) sPart[tw * kRowBlock + rt + lane] = make_float2(m, z);
    };
    if constexpr (ONE) {
      const int tok0 = u.tile0 * kTokPerWg + tw * kTokPerWave;
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();                      // the keys and the rows have landed
      bf16x8 kf[2][D / 16];
      load_key_frags<D>(sK + kTokPerWave * tw * (2 * D), qb0, kf);
#pragma unroll 1
      for (int rt = 32 * rg; rt < n_pad; rt += 32 * kRowGroups) {
        float m = -INFINITY, z = 0.f;
        if (tok0 < u.T) add_tokens(kf, rt, tok0, limit_of(rt), m, z);
        store(rt, m, z);
      }
    } else {
      float m_run[kTilesPerWave], z_run[kTilesPerWave];      // of row tile rg + 3 i
      int lim[kTilesPerWave];
#pragma unroll
      for (int i = 0; i < kTilesPerWave; ++i) {
        m_run[i] = -INFINITY;
        z_run[i] = 0.f;
        lim[i] = limit_of(32 * (rg + kRowGroups * i));
      }
      for (int tile = u.tile0; tile < u.tile1; ++tile) {
        const int tok0 = tile * kTokPerWg + tw * kTokPerWave;
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();                      // the tile's keys (and the rows) have landed
        bf16x8 kf[2][D / 16];
        load_key_frags<D>(sK + kTokPerWave * tw * (2 * D), qb0, kf);
        __syncthreads();                      // every wave has its keys
        if (tile + 1 < u.tile1) keys.load(tile + 1, wave);
        if (tok0 >= u.T) continue;
#pragma unroll
        for (int i = 0; i < kTilesPerWave; ++i) {
          const int rt = 32 * (rg + kRowGroups * i);
          if (rt < n_pad) add_tokens(kf, rt, tok0, lim[i], m_run[i], z_run[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < kTilesPerWave; ++i) {
        const int rt = 32 * (rg + kRowGroups * i);
        if (rt < n_pad) store(rt, m_run[i], z_run[i]);
      }
    }
    __syncthreads();
    // the four token slices' partials of a row fold, in slice order, into the unit's partial
    for (int r = tid; r < n_rows; r += kThreads) {
      float2 p[kTokWaves];
      float m = -INFINITY;
#pragma unroll
      for (int w = 0; w < kTokWaves; ++w) { p[w] = sPart[w * kRowBlock + r]; m = fmaxf(m, p[w].x); }
      float z = 0.f;
#pragma unroll
      for (int w = 0; w < kTokWaves; ++w)
        if (p[w].x > -INFINITY || (kPairs<D> && p[w].y != p[w].y)) z += p[w].y * exp2f((p[w].x - m) * kMaxScale<D>);
      const int rr = r_begin + r;
      const int i = rr / a.G, hh = rr - i * a.G;
      part[(p0 + i) * a.H + u.g * a.G + hh] = make_float2(m, z);
    }
  }
  if constexpr (RR) turned.store(rr, rot, a, u, sK);
}

// Folds a batch of (maximum, sumexp2) partials, in order, into the running pair (m, z).  A partial that saw
// nothing is (-inf, 0) and contributes 0 * exp2(-inf) = 0.
template <int D>
__device__ __forceinline__ void fold_partials(const float2 (&p)[kFoldBatch], float& m, float& z) {
  float mn = m;
#pragma unroll
  for (int u = 0; u < kFoldBatch; ++u) mn = fmaxf(mn, p[u].x);
  if (mn > -INFINITY) {
    z *= __builtin_amdgcn_exp2f((m - mn) * kMaxScale<D>);
#pragma unroll
    for (int u = 0; u < kFoldBatch; ++u) z = __builtin_fmaf(p[u].y, __builtin_amdgcn_exp2f((p[u].x - mn) * kMaxScale<D>), z);
    m = mn;
  }
}

// Pass 2, same division of work; the three row groups' column sums are added in a fixed order at the end of a tile.
template <int D, bool LIMIT, bool ONE>
__global__ __launch_bounds__(kThreads) void score_pass2(Args<ONE> pa) {
  const ScoreArgs& a = common(pa);
  extern __shared__ __align__(256) unsigned char smem[];      // (fragment addresses are formed with XORs below 256)
  unsigned char* sK = smem + kQBytes<D>;
  float* sL = reinterpret_cast<float*>(smem + kQBytes<D> + kKBytes<D>);          // [kRowBlock] maximum
  float* sRz = sL + kRowBlock;                                              // [kRowBlock] 1 / sum
  int* sLim = reinterpret_cast<int*>(sRz + kRowBlock);                      // [kRowBlock]
  float* sCol = reinterpret_cast<float*>(sLim + kRowBlock);                 // [kRowGroups][kTokPerWg]
  static_assert(kRowBlock <= kThreads, "one thread folds one staged row");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tw = wave % kTokWaves, rg = wave / kTokWaves;
  const uint32_t lds0 = lds_offset_of(smem);
  Unit u;
  if (!locate_unit(pa, u)) return;
  const int64_t p0 = min(max(a.probe_off[u.b], (int64_t)0), a.total_probe);
  const int64_t p1 = min(max(a.probe_off[u.b + 1], p0), a.total_probe);
  const int rows = (int)(p1 - p0) * a.G;
  if (rows == 0) return;                 // (the reduce kernel gives such a request zeros without reading the sums)
  const bf16_t* q = probes_of(pa, u);
  const KeyLoader<D> keys(keys_of(pa, u) + (u.c0 * a.Hkv + u.g) * D, a.Hkv, u.T, lds0 + (uint32_t)kQBytes<D>, wave, lane);
  const int64_t part_stride = a.total_probe * a.H;
  const int qb0 = frag_base<D>(lane);
  float* colsum = a.colsum + ((int64_t)u.layer * a.Hkv + u.g) * a.total_ctx + u.c0;

  float col0 = 0.f, col1 = 0.f;           // column sums of tokens tok0 + lane%32 and + 32 over this wave's row tiles
  for (int r_begin = 0; r_begin < rows; r_begin += kRowBlock) {
    const int n_rows = min(kRowBlock, rows - r_begin);
    const int n_pad = (n_rows + 31) & ~31;
    __syncthreads();
    if (ONE && r_begin == 0) keys.load(u.tile0, wave);
    stage_q_async<D>(a, q, p0, u.g, r_begin, n_rows, n_pad, lds0, wave, lane);
    if (!ONE) keys.load(u.tile0, wave);
    // maximum and sum of staged row tid over the request: the units' partials folded in order, kFoldBatch at a
    // time (all loads first, then one maximum and one rescaled sum); every workgroup of the request computes the
    // same values
    if (tid < n_pad) {
      float l = INFINITY;               // rows that do not exist or see nothing: exp2(logit - inf) = 0
      float rz = 0.f;
      int lim = 0;
      if (tid < n_rows) {
        const int rr = r_begin + tid, i = rr / a.G, hh = rr - i * a.G;
        const float2* pp = a.part + u.slot_first * part_stride + (p0 + i) * a.H + u.g * a.G + hh;
        float m = -INFINITY, z = 0.f;
        for (int t0 = 0; t0 < u.n_units; t0 += kFoldBatch) {
          float2 p[kFoldBatch];
#pragma unroll
          for (int v = 0; v < kFoldBatch; ++v)
            p[v] = (t0 + v < u.n_units) ? pp[v * part_stride] : make_float2(-INFINITY, 0.f);
          pp += kFoldBatch * part_stride;
          fold_partials<D>(p, m, z);
        }
        lim = LIMIT ? min(u.T, max(0, a.probe_limit[p0 + i])) : u.T;
        if (kPairs<D>) {
          if (lim > 0) {                // (no weight although tokens are visible, or a NaN sum: NaN)
            l = m;
            rz = z > 0.f ? 1.f / z : __builtin_nanf("");
          }
        } else if (z > 0.f) {
          l = m;
          rz = 1.f / z;
        }
      }
      sL[tid] = l;
      sRz[tid] = rz;
      sLim[tid] = lim;
    }
    for (int tile = u.tile0; tile < u.tile1; ++tile) {
      const int tok0 = tile * kTokPerWg + tw * kTokPerWave;
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();                    // the tile's keys (and the rows and their sums) have landed
      bf16x8 kf[2][D / 16];
      load_key_frags<D>(sK + kTokPerWave * tw * (2 * D), qb0, kf);
      if constexpr (!ONE) {
        __syncthreads();                  // every wave has its keys, and the previous tile's column sums are out
        if (tile + 1 < u.tile1) keys.load(tile + 1, wave);
        col0 = col1 = 0.f;
      }
      if (tok0 < u.T)
        for (int rt = 32 * rg; rt < n_pad; rt += 32 * kRowGroups) {
          floatx16 acc0, acc1;
          logit_tile<D, false>(kf, lds0 + (uint32_t)(rt * 2 * D + qb0), acc0, acc1);
          // lane owns tokens tok0 + lane%32 (acc0) and + 32 (acc1); register v is probe row
          // rt + 8*(v/4) + 4*(lane/32) + v%4
          const int tA = tok0 + (lane & 31), tB = tA + 32;
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const int rbase = rt + 8 * q4 + 4 * (lane >> 5);
            const float4 l4 = *reinterpret_cast<const float4*>(sL + rbase);
            const float4 z4 = *reinterpret_cast<const float4*>(sRz + rbase);
            const float ls[4] = {l4.x, l4.y, l4.z, l4.w};
            const float rz[4] = {z4.x, z4.y, z4.z, z4.w};
            int lims[4] = {u.T, u.T, u.T, u.T};
            if (LIMIT) {
              const int4 m4 = *reinterpret_cast<const int4*>(sLim + rbase);
              lims[0] = m4.x; lims[1] = m4.y; lims[2] = m4.z; lims[3] = m4.w;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const int v = 4 * q4 + c;
              float pa_ = exp_of<D>(acc0[v], ls[c]);
              float pb_ = exp_of<D>(acc1[v], ls[c]);
              if (LIMIT) {                 // (a row that sees nothing may have a NaN weight: the product first)
                pa_ = tA < lims[c] ? pa_ * rz[c] : 0.f;
                pb_ = tB < lims[c] ? pb_ * rz[c] : 0.f;
                col0 += pa_;
                col1 += pb_;
              } else {
                col0 = __builtin_fmaf(pa_, rz[c], col0);
                col1 = __builtin_fmaf(pb_, rz[c], col1);
              }
            }
          }
        }
      if (ONE && r_begin + kRowBlock < rows) continue;      // (the sums of all blocks of rows go out together)
      col0 += other_half(col0);
      col1 += other_half(col1);
      if (lane < 32) {
        float* sc = sCol + rg * kTokPerWg + tw * kTokPerWave;
        sc[lane] = col0;                      // (zero for a slice past the end of the request)
        sc[32 + lane] = col1;
      }
      __syncthreads();
      const int t = tile * kTokPerWg + tid;
      if (tid < kTokPerWg && t < u.T) {
        float sum = sCol[tid];
#pragma unroll
        for (int r3 = 1; r3 < kRowGroups; ++r3) sum += sCol[r3 * kTokPerWg + tid];
        if (!ONE && r_begin > 0) sum += colsum[t];    // (this thread's own sum over the rows before)
        colsum[t] = sum;
      }
    }
  }
}

// ------------------------------------------------------------------ single-kernel path
//
// When the whole launch is resident at once (one workgroup per compute unit, at most as many workgroups as
// compute units) and a KV group has at most kRowBlock probe rows, one kernel does everything.  A workgroup of
// eight waves owns a 256-token tile of one KV head; wave w keeps tokens 32w .. 32w+31 stationary and walks all
// row tiles.  It keeps, in registers, e = 2^(logit - m) against the maximum m of its own 32 tokens for every
// (token, row) pair of the tile: the second exponential of a two-pass scheme becomes one multiply-add by
// 2^(m - lse) once the row's log-sum-exp over the whole request is known.
//
// Two hand-offs between workgroups, both through device-scope relaxed atomics on data that is itself written
// and read with device-scope atomic stores and loads (they bypass the non-coherent caches; a wave waits for
// its own stores to complete before it signals, so no cache-wide release or acquire fence is needed):
//   1. the tiles of one (request, KV head) exchange their per-row (max, sum-exp): every workgroup publishes
//      its partials, adds one to the group's arrival counter and waits until all tiles of the request have
//      arrived (bounded wait: all workgroups of the launch are resident, so every one of them is running);
//   2. the KV heads of one tile exchange their column sums: the last head to arrive (found with a counter; no
//      waiting) adds the heads in head order and writes the scores.
// All sums run in a fixed order, so the scores are bit-stable.  The counters live in a device array that the
// loader zero-fills; the last workgroup to finish resets the ones this launch used, so every launch starts from
// zero without a clearing kernel.  Launches take turns over kSyncSlots sets of counters.

constexpr int kFusedWaves = 8;
constexpr int kFusedThreads = 64 * kFusedWaves;
constexpr int kFusedRowTiles = kRowBlock / 32;
constexpr int kSyncSlots = 8;
constexpr uint32_t kSpinLimit = 1u << 20;  // polls (a microsecond or two each) before a workgroup gives up waiting

__device__ uint32_t g_sync[kSyncSlots * kSyncWords];

struct FusedArgs {
  ScoreArgs s;
  float2* part;        // [tile][Hkv][kRowBlock] (max2, sumexp2) of the tile, published with atomic stores
  float* colpart;      // [tile][Hkv][kTokPerWg] column sums of one KV head
  uint32_t* sync;      // this launch's counter slot
  int n_wg_tiles;      // tiles the grid provides (upper bound on the tiles of all requests)
  uint32_t spin_limit;
  Rerotation r;
};

__device__ __forceinline__ void publish(float2* p, float2 v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, v), __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 fetch(const float2* p) {
  return __builtin_bit_cast(float2, __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void publish(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float fetch(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr size_t kFusedLds = kQBytes<128> + kKBytes<128>;
// Re-rotation of a tile (RR): the chunk table, each row's chunk, and the (cos, sin) pairs of the tile's chunks, behind the
// staged rows.
constexpr int kRotChunks = 8;                     // chunks whose pairs are kept at a time
static_assert(kRotChunksPerTile == 2 * kRotChunks, "two fillings to a tile, on average");
struct RotLds {
  qcf_chunk table[kMaxRotChunks];
  const char* k[kTokPerWg];                       // source of a row, for this KV head (row of no chunk: itself)
  const char* v[kTokPerWg];
  int chunk[kTokPerWg];                           // of a row, -1: none
  float2 cs[kRotChunks * 64];
};
constexpr size_t kFusedRotLds = kFusedLds + sizeof(RotLds);
static_assert(kFusedRotLds + 1024 <= 160 * 1024, "one workgroup's LDS");

__device__ __forceinline__ bf16x8 pack8(const float* o) {
  return __builtin_bit_cast(bf16x8, mk4(cvt_pk_bf16(o[0], o[1]), cvt_pk_bf16(o[2], o[3]), cvt_pk_bf16(o[4], o[5]), cvt_pk_bf16(o[6], o[7])));
}
// Turns the key fragments of a lane's row by the pairs at cs: element e of fragment ks is 16 ks + 8 hf + e of the row.
__device__ __forceinline__ void turn_frags(bf16x8 (&kf)[8], const float2* cs, int hf, bool interleaved) {
  if (!interleaved) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      float f[16], o[16];
      Vec16<bf16_t>::unpack(__builtin_bit_cast(u32x4, kf[ks]), f);
      Vec16<bf16_t>::unpack(__builtin_bit_cast(u32x4, kf[ks + 4]), f + 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) turn_pair(f[e], f[e + 8], cs[16 * ks + 8 * hf + e], o[e], o[e + 8]);
      kf[ks] = pack8(o);
      kf[ks + 4] = pack8(o + 8);
    }
  } else {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      float f[8], o[8];
      Vec16<bf16_t>::unpack(__builtin_bit_cast(u32x4, kf[ks]), f);
#pragma unroll
      for (int e = 0; e < 8; e += 2) turn_pair(f[e], f[e + 1], cs[8 * ks + 4 * hf + e / 2], o[e], o[e + 1]);
      kf[ks] = pack8(o);
    }
  }
}

// RR: the keys of the tile come from the chunk caches, are turned to their global positions in the registers that score them
// and written to the fused cache from there; the values are copied while the first hand-off is on its way.  Saves the launch of qcf_rerope,
// its pass over the cache and the reading of the keys.  Re-rotation and scoring, us, in two launches and in one: 731 tokens, 96
// rows of a group 5.7 + 13.9 and 18.9; 4096, 160 rows 8.6 + 17.3 and 22.6; 8192, 320 rows 13.8 + 27.4 and 34.7.  Everything in
// front of the keys' loads is a chain of latencies (with the rows' sources looked up by every use of them 19.7, 23.8 and 36.9;
// with the values prefetched into the L2 as well 22.2, 26.0 and 37.5; copied in front of the first hand-off, which then waits
// for their stores, 23.4, 28.5 and 42.0).
template <bool LIMIT, bool RR>
__global__ __launch_bounds__(kFusedThreads) void score_fused(FusedArgs fa) {
  constexpr int D = 128;
  const ScoreArgs& a = fa.s;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* sK = smem + kQBytes<D>;
  // (reused once the key fragments are in registers)
  float2* sPart = reinterpret_cast<float2*>(sK);                            // [kFusedWaves][kRowBlock]
  float* sL = reinterpret_cast<float*>(sK + kFusedWaves * kRowBlock * 8);   // [kRowBlock] log2-sum-exp
  float* sCol = sL + kRowBlock;                                             // [kTokPerWg]
  __shared__ int s_flag[2];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5, l32 = lane & 31;
  const int g = (int)(blockIdx.x % a.Hkv);
  const int wg_tile = (int)(blockIdx.x / a.Hkv);
  const int n_wg = fa.n_wg_tiles * a.Hkv;

  RotLds& rot = *reinterpret_cast<RotLds*>(smem + kFusedLds);  // (RR)
  if constexpr (RR)
    for (int i = tid; i < fa.r.n_chunks * (int)(sizeof(qcf_chunk) / 8); i += kFusedThreads)
      reinterpret_cast<uint64_t*>(rot.table)[i] = reinterpret_cast<const uint64_t*>(fa.r.chunks)[i];
  int b, T, tile_tok0, tile_first;
  int64_t c0;
  const bool have_tile = locate_tile(a, wg_tile, b, c0, T, tile_tok0, tile_first);
  int rows = 0;
  int64_t p0 = 0;
  if (have_tile) {
    p0 = min(max(a.probe_off[b], (int64_t)0), a.total_probe);
    const int64_t p1 = min(max(a.probe_off[b + 1], p0), a.total_probe);
    rows = min((int)(p1 - p0) * a.G, kRowBlock);       // (the launcher only takes this path when all rows fit)
  }
  const int n_tiles = have_tile ? (T + kTokPerWg - 1) / kTokPerWg : 0;
  const int n_rt = (rows + 31) >> 5;
  constexpr float k2 = kK2<D>;
  constexpr int KS = D / 16;

  float e[kFusedRowTiles][16];      // 2^(logit - m_w) of (token, row) pairs; row = 32 rt + l32
  bf16x8 kf[KS];
  const int fb0 = frag_base<D>(lane);
  const int64_t row_elems = (int64_t)a.Hkv * D, tile_row0 = c0 + tile_tok0;      // (RR) of the cache
  auto copy_values = [&]() {
    constexpr int kPer = kFusedThreads / 16, kVals = kTokPerWg / kPer;           // rows at a time, 16-byte vectors per thread
    u32x4 vals[kVals];
#pragma unroll
    for (int p = 0; p < kVals; ++p) vals[p] = *reinterpret_cast<const u32x4*>(rot.v[p * kPer + (tid >> 4)] + (tid & 15) * 16);
    bf16_t* dst = fa.r.v + (tile_row0 + (tid >> 4)) * row_elems + g * D + (tid & 15) * 8;
#pragma unroll
    for (int p = 0; p < kVals; ++p)
      if (tile_tok0 + p * kPer + (tid >> 4) < T) *reinterpret_cast<u32x4*>(dst + p * kPer * row_elems) = vals[p];
  };

  if (rows > 0 || (RR && have_tile)) {
    if constexpr (RR) {
      __syncthreads();                                  // the table is there
      if (tid < kTokPerWg) {
        const int64_t row = c0 + min(tile_tok0 + tid, T - 1);
        const int c = chunk_of(rot.table, fa.r.n_chunks, row);
        const qcf_chunk& ch = rot.table[c];
        const bool covered = row >= ch.dst_row && row < ch.dst_row + ch.len;
        const int64_t off = ((covered ? row - ch.dst_row : row) * row_elems + g * D) * 2;
        rot.k[tid] = static_cast<const char*>(covered ? ch.k_src : fa.r.k) + off;
        rot.v[tid] = static_cast<const char*>(covered ? ch.v_src : fa.r.v) + off;
        rot.chunk[tid] = covered ? c : -1;
      }
      __syncthreads();
    }
    constexpr int kKeyLoads = kTokPerWg / kRowsPerLoad<D> / kFusedWaves;         // keys
    const char* key_src[kKeyLoads];
#pragma unroll
    for (int i = 0; i < kKeyLoads; ++i) {
      const int r = staged_row<D>(wave + i * kFusedWaves, lane);
      if constexpr (RR) key_src[i] = rot.k[r] + staged_elem<D>(r, lane) * 2;
      else key_src[i] = reinterpret_cast<const char*>(a.k + ((c0 + min(tile_tok0 + r, T - 1)) * a.Hkv + g) * D + staged_elem<D>(r, lane));
    }
#pragma unroll
    for (int i = 0; i < kKeyLoads; ++i) load_to_lds_addr(key_src[i], sK + (wave + i * kFusedWaves) * 1024);
    for (int j = wave; j < n_rt * (32 / kRowsPerLoad<D>); j += kFusedWaves) {    // probe rows of the group
      const int r = staged_row<D>(j, lane);
      const int rr = min(r, rows - 1);
      const int i = rr / a.G, hh = rr - i * a.G;
      load_to_lds_addr(a.q + ((p0 + i) * a.H + g * a.G + hh) * D + staged_elem<D>(r, lane), smem + j * 1024);
    }
    int first_chunk = 0, n_mine = 0;                    // (RR) chunks from the tile's first row to its last
    auto fill_pairs = [&](int from) {                   // pairs of the tile's chunks from .. from + kRotChunks - 1
      for (int i = tid; i < min(kRotChunks, n_mine - from) * 64; i += kFusedThreads)
        rot.cs[i] = shift_pair(rot.table[first_chunk + from + i / 64], fa.r.neg2_over_d_log2base, i % 64);
    };
    if constexpr (RR) {
      first_chunk = chunk_of(rot.table, fa.r.n_chunks, tile_row0);
      n_mine = chunk_of(rot.table, fa.r.n_chunks, c0 + min(tile_tok0 + kTokPerWg, T) - 1) - first_chunk + 1;
      fill_pairs(0);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      kf[ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(sK + (32 * wave) * (2 * D) + (fb0 ^ (32 * ks))));
    if constexpr (RR) {
      const int mine = rot.chunk[32 * wave + l32] - first_chunk;        // (negative: not turned)
      for (int from = 0;; from += kRotChunks) {
        if (mine >= from && mine < from + kRotChunks) turn_frags(kf, rot.cs + (mine - from) * 64, hf, fa.r.style != 0);
        if (from + kRotChunks >= n_mine) break;
        __syncthreads();
        fill_pairs(from + kRotChunks);
        __syncthreads();
      }
      if (tile_tok0 + 32 * wave + l32 < T) {
        bf16_t* dst = fa.r.k + (tile_row0 + 32 * wave + l32) * row_elems + g * D + 8 * hf;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) *reinterpret_cast<u32x4*>(dst + 16 * ks) = __builtin_bit_cast(u32x4, kf[ks]);
      }
      if (rows == 0) copy_values();
    }
  }
  if constexpr (RR) {                                   // rows of the cache outside the request (none, as a rule)
    const int64_t lo = min(max(a.ctx_off[0], (int64_t)0), a.total_ctx), hi = min(max(a.ctx_off[1], lo), a.total_ctx);
    if (hi - lo < a.total_ctx) {
      __syncthreads();                                  // (the table, where no tile has waited for it)
      for (int64_t i = wg_tile * kFusedWaves + wave; i < a.total_ctx - (hi - lo); i += fa.n_wg_tiles * kFusedWaves)
        rerotate_row<128>(fa.r, rot.table, i < lo ? i : i + (hi - lo), a.Hkv, g, lane);
    }
  }
  if (rows > 0) {
    // probe-row fragments travel through a ring of four registers: the fragment four further (of this tile or
    // the next) is requested right behind the MFMA that used the slot.  One address register per
    // fragment index; the row tile is a constant offset of the read.
    uint32_t qaddr[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qaddr[ks] = lds_offset_of(smem) + (uint32_t)(fb0 ^ (32 * ks));
    auto qfrag = [&](int rt, int ks) {
      return *(const u32x4 __attribute__((address_space(3)))*)(uintptr_t)(qaddr[ks] + (uint32_t)(rt * 32 * 2 * D));
    };
    u32x4 ring[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) ring[i] = qfrag(0, i);
    __syncthreads();                               // the key tile's LDS is reused from here on
    const int tok0 = tile_tok0 + 32 * wave;
#pragma unroll
    for (int rt = 0; rt < kFusedRowTiles; ++rt) {
      if (rt < n_rt) {
        floatx16 acc = {0};
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
          // S^T tile: rows = tokens (A = keys), columns = probe rows (B = queries)
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], __builtin_bit_cast(bf16x8, ring[ks & 3]), acc, 0, 0, 0);
          if (ks + 4 < KS) ring[ks & 3] = qfrag(rt, ks + 4);
          else if (rt + 1 < kFusedRowTiles) ring[ks & 3] = qfrag(rt + 1, ks + 4 - KS);   // (unused after the last tile)
        }
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {          // issue order: every read sits behind the MFMA that frees its slot
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (ks + 4 < KS || rt + 1 < kFusedRowTiles) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        // lane owns probe row 32 rt + l32; register v is token tok0 + 8 (v/4) + 4 hf + v%4
        float sv[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) sv[v] = acc[v];
        if (LIMIT || tok0 + 32 > T) {            // wave-uniform: only ragged or limited tiles compare
          const int r = 32 * rt + l32;
          int lim = T;
          if (LIMIT && r < rows) lim = min(T, max(0, a.probe_limit[p0 + r / a.G]));
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int t0 = tok0 + 8 * (v >> 2) + 4 * hf + (v & 3);
            sv[v] = (t0 < lim) ? sv[v] : -INFINITY;
          }
        }
        float mx = sv[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, sv[v]);
        mx = fmaxf(mx, other_half(mx)) * k2;          // k2 > 0: scaling commutes with the maximum
        const float m_use = (mx == -INFINITY) ? 0.f : mx;
        float sum = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          e[rt][v] = __builtin_amdgcn_exp2f(__builtin_fmaf(sv[v], k2, -m_use));
          sum += e[rt][v];
        }
        sum += other_half(sum);
        if (lane < 32) sPart[wave * kRowBlock + 32 * rt + lane] = make_float2(mx, sum);
      } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) e[rt][v] = 0.f;
      }
    }
    __syncthreads();
    // the eight token slices' partials of a row fold, in slice order, into the tile's partial
    float2* part = fa.part + ((int64_t)wg_tile * a.Hkv + g) * kRowBlock;
    for (int r = tid; r < rows; r += kFusedThreads) {
      float2 p[kFusedWaves];
      float m = -INFINITY;
#pragma unroll
      for (int w = 0; w < kFusedWaves; ++w) { p[w] = sPart[w * kRowBlock + r]; m = fmaxf(m, p[w].x); }
      float z = 0.f;
#pragma unroll
      for (int w = 0; w < kFusedWaves; ++w)
        if (p[w].x > -INFINITY) z += p[w].y * exp2f(p[w].x - m);
      publish(part + r, make_float2(m, z));
    }
    __builtin_amdgcn_s_waitcnt(0);            // this thread's partials have reached memory
    __syncthreads();
    // hand-off 1: the tiles of (request b, KV head g)
    uint32_t* cnt = fa.sync + 1 + b * a.Hkv + g;
    if (tid == 0) __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if constexpr (RR) copy_values();                   // (not earlier: the partials would wait for its stores)
    if (tid == 0) {
      uint32_t spins = 0;
      while (__hip_atomic_load(cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (uint32_t)n_tiles &&
             ++spins < fa.spin_limit)
        __builtin_amdgcn_s_sleep(1);
    }
    __syncthreads();
    // log2-sum-exp of row r over the request: the tiles' partials folded in tile order (up to 32 loads in
    // flight per thread)
    for (int r = tid; r < rows; r += kFusedThreads) {
      const float2* pp = fa.part + ((int64_t)tile_first * a.Hkv + g) * kRowBlock + r;
      const int64_t stride = (int64_t)a.Hkv * kRowBlock;
      float m = -INFINITY, z = 0.f;
      for (int t0 = 0; t0 < n_tiles; t0 += 2 * kFoldBatch) {
        float2 pa[kFoldBatch], pb[kFoldBatch];
#pragma unroll
        for (int u = 0; u < kFoldBatch; ++u) {
          pa[u] = (t0 + u < n_tiles) ? fetch(pp + u * stride) : make_float2(-INFINITY, 0.f);
          pb[u] = (t0 + kFoldBatch + u < n_tiles) ? fetch(pp + (kFoldBatch + u) * stride) : make_float2(-INFINITY, 0.f);
        }
        pp += 2 * kFoldBatch * stride;
        fold_partials<D>(pa, m, z);
        fold_partials<D>(pb, m, z);
      }
      sL[r] = (z > 0.f) ? m + log2f(z) : INFINITY;      // a row that sees nothing: every weight is 0
    }
    for (int r = rows + tid; r < 32 * n_rt; r += kFusedThreads) sL[r] = INFINITY;
    __syncthreads();
    // column sums over this wave's rows: e * 2^(m_w - lse), row tiles in order, then over the lanes
    float col[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) col[v] = 0.f;
#pragma unroll
    for (int rt = 0; rt < kFusedRowTiles; ++rt) {
      if (rt < n_rt) {
        const float l = sL[32 * rt + l32];
        const float mw = sPart[wave * kRowBlock + 32 * rt + l32].x;
        const float w = (mw == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(mw - l);
#pragma unroll
        for (int v = 0; v < 16; ++v) col[v] = __builtin_fmaf(e[rt][v], w, col[v]);
      }
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) col[v] = half_wave_sum(col[v]);
    if (l32 == 0) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sCol[32 * wave + 8 * (v >> 2) + 4 * hf + (v & 3)] = col[v];
    }
    __syncthreads();
    float* colpart = fa.colpart + ((int64_t)wg_tile * a.Hkv + g) * kTokPerWg;
    if (tid < kTokPerWg) publish(colpart + tid, sCol[tid]);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    // hand-off 2: the KV heads of this tile; the last one to arrive adds them up.  The count of finished
    // workgroups is sent right behind (its operand depends on the first counter's answer, so the two
    // additions cannot pass each other) and its answer is only looked at after the sums.
    uint32_t fin = 0;
    if (tid == 0) {
      uint32_t* cnt = fa.sync + 1 + a.B * a.Hkv + wg_tile;
      const uint32_t old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_flag[0] = (old == (uint32_t)a.Hkv - 1u) ? 1 : 0;
      fin = __hip_atomic_fetch_add(fa.sync, 1u + (old >> 31), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (s_flag[0] && tid < kTokPerWg && tile_tok0 + tid < T) {
      const float* cp = fa.colpart + (int64_t)wg_tile * a.Hkv * kTokPerWg + tid;
      float acc = 0.f;
      for (int gg = 0; gg < a.Hkv; ++gg) acc += fetch(cp + gg * kTokPerWg);
      write_score(a, c0 + tile_tok0 + tid, acc / (float)((rows / a.G) * a.H));
    }
    if (tid == 0) s_flag[1] = (fin == (uint32_t)n_wg - 1u) ? 1 : 0;
    __syncthreads();
  } else {
    // a request without probe rows scores zero everywhere
    if (have_tile && g == 0 && tid < kTokPerWg && tile_tok0 + tid < T) write_score(a, c0 + tile_tok0 + tid, 0.f);
    if (tid == 0) {
      const uint32_t fin = __hip_atomic_fetch_add(fa.sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_flag[1] = (fin == (uint32_t)n_wg - 1u) ? 1 : 0;
    }
    __syncthreads();
  }
  // the last workgroup of the launch to have counted itself finished puts the launch's counters back to zero
  // (every other workgroup has used its counters by then: a workgroup counts itself after its last use)
  if (s_flag[1]) {
    const int n_words = 1 + a.B * a.Hkv + fa.n_wg_tiles;
    for (int i = tid; i < n_words; i += kFusedThreads)
      __hip_atomic_store(fa.sync + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Adds the KV heads of every layer in order, and the layers, in order, into the score.  Several layers: layers_at a time by as
// many groups of threads, 256 / layers_at tokens to a workgroup, so that the loads of all of them are on their way together (8
// layers of 6001 tokens, 24 workgroups with one layer after the other: 6.4 us, now 4.6).
__host__ __device__ __forceinline__ int layers_at(int n_layers) { return n_layers >= 4 ? 4 : n_layers >= 2 ? 2 : 1; }
template <bool ONE>
__global__ __launch_bounds__(256) void score_reduce(Args<ONE> pa) {
  const ScoreArgs& a = common(pa);
  __shared__ float s_sum[ONE ? 1 : kMaxLayers * 256 / 4];        // [layer][token]
  int at = 1;
  if constexpr (!ONE) at = layers_at(pa.n_layers);
  const int toks = 256 / at, tok = (int)threadIdx.x % toks;
  const int64_t j = (int64_t)blockIdx.x * toks + tok;
  const int b = j < a.total_ctx ? find_request(a.ctx_off, a.B, j) : a.B;
  int64_t p0 = 0, p1 = 0;
  if (b < a.B) {
    p0 = min(max(a.probe_off[b], (int64_t)0), a.total_probe);
    p1 = min(max(a.probe_off[b + 1], p0), a.total_probe);
  }
  const float n = (float)((p1 - p0) * a.H);
  if constexpr (ONE) {
    if (b >= a.B) return;
    float acc = 0.f;
    for (int g = 0; g < a.Hkv; ++g) acc += a.colsum[(int64_t)g * a.total_ctx + j];
    write_score(a, j, p1 > p0 ? acc / n : 0.f);
  } else {
    auto layer_sum = [&](int l) {
      const float* col = a.colsum + (int64_t)l * a.Hkv * a.total_ctx + j;
      float acc = 0.f;
#pragma unroll 8
      for (int g = 0; g < a.Hkv; ++g) acc += col[g * a.total_ctx];
      return p1 > p0 ? acc / n : 0.f;
    };
    float score = b < a.B && a.beta != 0.f ? a.score[j] : 0.f;
    if (at == 1) {
      if (b < a.B) a.score[j] = blended(a.beta, score, pa.alpha[0] * layer_sum(0));
      return;
    }
    if (b < a.B)
#pragma unroll 2
      for (int l = (int)threadIdx.x / toks; l < pa.n_layers; l += at) s_sum[l * toks + tok] = layer_sum(l);
    __syncthreads();
    if ((int)threadIdx.x >= toks || b >= a.B) return;
    for (int l = 0; l < pa.n_layers; ++l) score = blended(l == 0 ? a.beta : 1.f, score, pa.alpha[l] * s_sum[l * toks + tok]);
    a.score[j] = score;
  }
}

__global__ __launch_bounds__(256) void score_zero(float* score, int64_t n, float beta) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j < n) score[j] = (beta == 0.f) ? 0.f : beta * score[j];
}

template <int D> constexpr size_t kPass2Lds = kQBytes<D> + kKBytes<D> + kRowBlock * 4 * 3 + (size_t)kRowGroups * kTokPerWg * sizeof(float);
static_assert((size_t)kFusedWaves * kRowBlock * 8 + (size_t)kRowBlock * 4 + (size_t)kTokPerWg * 4 <= kKBytes<128>,
              "the single-kernel path's tables fit in the key tile's LDS");

template <bool LIMIT, bool RR>
qcf_status run_fused(const FusedArgs& fa, hipStream_t st) {
  static std::atomic<uint64_t> lds_ok;
  constexpr size_t lds = RR ? kFusedRotLds : kFusedLds;
  QCF_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(&score_fused<LIMIT, RR>), lds, lds_ok));
  score_fused<LIMIT, RR><<<dim3((unsigned)(fa.n_wg_tiles * fa.s.Hkv)), dim3(kFusedThreads), lds, st>>>(fa);
  return check_launch("score (single kernel)");
}

template <int D, bool LIMIT, bool ONE, bool RR = false>
qcf_status run_two_pass(const Args<ONE>& a, dim3 grid, hipStream_t st, bool reduce, const RerotationOf<RR>& r = {}) {
  static std::atomic<uint64_t> lds_ok[2];
  constexpr size_t lds = kPass1Lds<D> + (RR ? sizeof(Pass1Rot) : 0);
  static_assert(lds + 1024 <= 160 * 1024, "one workgroup's LDS");
  QCF_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(&score_pass1<D, LIMIT, ONE, RR>), lds, lds_ok[0]));
  QCF_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(&score_pass2<D, LIMIT, ONE>), kPass2Lds<D>, lds_ok[1]));
  const dim3 block(kThreads);
  score_pass1<D, LIMIT, ONE, RR><<<grid, block, lds, st>>>(a, r);
  QCF_TRY_LAUNCH("score pass 1");
  score_pass2<D, LIMIT, ONE><<<grid, block, kPass2Lds<D>, st>>>(a);
  QCF_TRY_LAUNCH("score pass 2");
  if (!reduce) return QCF_OK;
  int toks = 256;
  if constexpr (!ONE) toks /= layers_at(a.n_layers);
  score_reduce<ONE><<<dim3((unsigned)((common(a).total_ctx + toks - 1) / toks)), dim3(256), 0, st>>>(a);
  return check_launch("score reduce");
}
template <bool ONE>
qcf_status run_passes(int D, const Args<ONE>& a, dim3 grid, hipStream_t st, bool reduce) {
  const bool limit = common(a).probe_limit != nullptr;
  if (D == 128) return limit ? run_two_pass<128, true, ONE>(a, grid, st, reduce) : run_two_pass<128, false, ONE>(a, grid, st, reduce);
  return limit ? run_two_pass<64, true, ONE>(a, grid, st, reduce) : run_two_pass<64, false, ONE>(a, grid, st, reduce);
}

// The two passes over n_layers layers (up to kMaxLayers); a: everything but the layers and the workspace.
qcf_status launch_two_pass(const qcf_layer_desc& L, const ScoreArgs& a, int n_layers, const void* const* q,
                           const void* const* k, const float* alpha, void* ws, hipStream_t st, ScoreSums* left = nullptr,
                           const Rerotation* r = nullptr) {
  const PassWs w = pass_ws(L, n_layers, a.B, a.total_probe, a.total_ctx);
  // (nothing has been enqueued: a call that asks for a re-rotation which this would leave out must not go on without it)
  if (r && !pass1_rerotates(L, w.unit_tiles, n_layers, a.probe_limit != nullptr))
    return fail(QCF_ERR_UNSUPPORTED, "score: no re-rotation in units of %d tiles, %d layers, heads of %d", w.unit_tiles, n_layers, L.head_dim);
  if (w.n_units * n_layers * a.Hkv > 0x7fffffff) return fail(QCF_ERR_UNSUPPORTED, "score: grid too large");
  PassArgs pa;
  pa.s = a;
  pa.s.part = static_cast<float2*>(ws);
  pa.s.colsum = reinterpret_cast<float*>(static_cast<char*>(ws) + w.colsum);
  for (int l = 0; l < kMaxLayers; ++l) {
    const int i = std::min(l, n_layers - 1);
    pa.q[l] = static_cast<const bf16_t*>(q[i]);
    pa.k[l] = static_cast<const bf16_t*>(k[i]);
    pa.alpha[l] = alpha[i];
  }
  pa.n_layers = n_layers;
  pa.unit_tiles = w.unit_tiles;
  pa.unit_magic = (uint32_t)((1ull << 32) / (unsigned)w.unit_tiles + 1);       // (a request has at most 2^22 tiles, a unit 64)
  pa.n_units = (int)w.n_units;
  if (left) *left = ScoreSums{pa.s.colsum, a.probe_off, a.total_probe, a.H, a.Hkv, false};
  if (n_layers > 1 || w.unit_tiles > 1 || a.Hkv > 65535)
    return run_passes<false>(L.head_dim, pa, dim3((unsigned)(w.n_units * n_layers * a.Hkv)), st, !left);
  const dim3 grid((unsigned)w.n_units, (unsigned)a.Hkv);
  if (r) return run_two_pass<64, false, true, true>(pa.s, grid, st, !left, *r);
  return run_passes<true>(L.head_dim, pa.s, grid, st, !left);
}

ScoreArgs score_args(const qcf_layer_desc& L, int32_t B, const void* q, const int64_t* probe_off, int64_t total_probe,
                     const void* k, const int64_t* ctx_off, int64_t total_ctx, const int32_t* probe_limit, float* score,
                     float alpha, float beta) {
  ScoreArgs a;
  a.q = static_cast<const bf16_t*>(q);
  a.k = static_cast<const bf16_t*>(k);
  a.probe_off = probe_off;
  a.ctx_off = ctx_off;
  a.probe_limit = probe_limit;
  a.total_probe = total_probe;
  a.total_ctx = total_ctx;
  a.B = B; a.H = L.n_q_heads; a.Hkv = L.n_kv_heads; a.G = a.H / a.Hkv;
  a.part = nullptr;
  a.colsum = nullptr;
  a.score = score;
  a.alpha = alpha;
  a.beta = beta;
  return a;
}

// Device address of the zero-initialised counter array on the current device (asked for once per device).
qcf_status sync_counters(uint32_t** out) {
  constexpr int kMaxDev = 64;
  static std::atomic<uint32_t*> ptr[kMaxDev];
  int dev = 0;
  QCF_TRY(check_hip(hipGetDevice(&dev), "hipGetDevice"));
  if (dev < 0 || dev >= kMaxDev) return fail(QCF_ERR_UNSUPPORTED, "device id %d >= %d", dev, kMaxDev);
  uint32_t* p = ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    void* q = nullptr;
    QCF_TRY(check_hip(hipGetSymbolAddress(&q, HIP_SYMBOL(g_sync)), "hipGetSymbolAddress(g_sync)"));
    if (!q) return fail(QCF_ERR_HIP, "hipGetSymbolAddress(g_sync) returned a null address");
    p = static_cast<uint32_t*>(q);
    ptr[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return QCF_OK;
}

// the arguments of a single-kernel launch, with the next set of counters
qcf_status fused_args(const qcf_layer_desc& L, const ScoreArgs& a, void* ws, FusedArgs* fa) {
  const FusedWs fw = fused_ws(L, a.B, a.total_ctx);
  *fa = FusedArgs{};
  fa->s = a;
  fa->part = reinterpret_cast<float2*>(static_cast<char*>(ws) + fw.part);
  fa->colpart = reinterpret_cast<float*>(static_cast<char*>(ws) + fw.colpart);
  fa->n_wg_tiles = (int)n_tiles_upper(a.B, a.total_ctx);
  fa->spin_limit = kSpinLimit;
  uint32_t* counters = nullptr;
  QCF_TRY(sync_counters(&counters));
  static std::atomic<uint32_t> next_slot{0};
  fa->sync = counters + (size_t)(next_slot.fetch_add(1, std::memory_order_relaxed) % kSyncSlots) * kSyncWords;
  return QCF_OK;
}

}  // namespace

qcf_status launch_rerope_score(const qcf_layer_desc& L, const qcf_chunk* chunks, int32_t n_chunks, const void* q,
                               const int64_t* probe_off, int64_t total_probe, void* k, void* v, const int64_t* ctx_off,
                               int64_t total_ctx, float* score, void* ws, hipStream_t st, ScoreSums* left) {
  const ScoreArgs a = score_args(L, 1, q, probe_off, total_probe, k, ctx_off, total_ctx, nullptr, score, 1.f, 0.f);
  const Rerotation r{chunks, n_chunks, L.rope_style, -2.0 / (double)L.head_dim * std::log2(L.rope_base), static_cast<bf16_t*>(k),
                     static_cast<bf16_t*>(v)};
  if (!use_fused(L, 1, total_probe, total_ctx)) {
    const void* keys = k;
    const float alpha = 1.f;
    return launch_two_pass(L, a, 1, &q, &keys, &alpha, ws, st, left, &r);
  }
  FusedArgs fa;
  QCF_TRY(fused_args(L, a, ws, &fa));
  fa.r = r;
  return run_fused<false, true>(fa, st);
}

qcf_status launch_score(const qcf_layer_desc& L, int32_t B, const void* q, const int64_t* probe_off,
                        int64_t total_probe, const void* k, const int64_t* ctx_off, int64_t total_ctx,
                        const int32_t* probe_limit, float* score, float alpha, float beta, void* ws, hipStream_t st, ScoreSums* left) {
  const int H = L.n_q_heads, Hkv = L.n_kv_heads, D = L.head_dim;
  if (total_probe == 0) {      // no probe rows at all: every score is 0 (no workspace was asked for)
    const int64_t blocks = (total_ctx + 255) / 256;
    score_zero<<<dim3((unsigned)blocks), dim3(256), 0, st>>>(score, total_ctx, beta);
    return check_launch("score zero");
  }
  const bool fused = use_fused(L, B, total_probe, total_ctx);
  if (!fused && !use_two_pass(L, B, total_probe, total_ctx)) {
    float* P = static_cast<float*>(ws);
    const int64_t col_blocks = (total_ctx + kColTokens - 1) / kColTokens;
    if (total_probe * H > 0x7fffffff || col_blocks > 0x7fffffff)
      return fail(QCF_ERR_UNSUPPORTED, "score: too many rows");
    if (total_probe > 0) {
      const dim3 grid((unsigned)(total_probe * H));
      const bool few = B > 1 && total_ctx <= (int64_t)kShortTokens * B;
#define QCF_ROWS_OF(T, DIM, THREADS)                                                                                  \
  score_rows_generic<T, DIM, THREADS><<<grid, dim3(THREADS), 0, st>>>(static_cast<const T*>(q), probe_off, total_probe, \
                                                                      static_cast<const T*>(k), ctx_off, total_ctx, B, probe_limit, H, Hkv, P)
#define QCF_ROWS(T, DIM) { if (few) QCF_ROWS_OF(T, DIM, 256); else QCF_ROWS_OF(T, DIM, 512); }
      if (L.dtype == QCF_DTYPE_BF16) {
        if (D == 64) QCF_ROWS(bf16_t, 64) else QCF_ROWS(bf16_t, 128)
      } else {
        if (D == 64) QCF_ROWS(float, 64) else QCF_ROWS(float, 128)
      }
#undef QCF_ROWS
#undef QCF_ROWS_OF
      QCF_TRY_LAUNCH("score rows");
    }
    if (left) {
      *left = ScoreSums{P, probe_off, total_probe, H, Hkv, true};
      return QCF_OK;
    }
    score_colmean_generic<<<dim3((unsigned)col_blocks), dim3(64 * kColWaves), 0, st>>>(P, probe_off, total_probe, ctx_off,
                                                                           total_ctx, B, H, score, alpha, beta);
    return check_launch("score column mean");
  }

  const ScoreArgs a = score_args(L, B, q, probe_off, total_probe, k, ctx_off, total_ctx, probe_limit, score, alpha, beta);
  if (fused) {
    FusedArgs fa;
    QCF_TRY(fused_args(L, a, ws, &fa));
    return probe_limit ? run_fused<true, false>(fa, st) : run_fused<false, false>(fa, st);
  }
  return launch_two_pass(L, a, 1, &q, &k, &alpha, ws, st, left);
}

// ---- several layers --------------------------------------------------------------------------------
qcf_status launch_score_layers(const qcf_layer_desc& L, int32_t n_layers, int32_t B, const void* const* q,
                               const int64_t* probe_off, int64_t total_probe, const void* const* k, const int64_t* ctx_off,
                               int64_t total_ctx, const int32_t* probe_limit, const float* weights, float* score, void* ws,
                               hipStream_t st) {
  const int at_once = layers_at_once(L, n_layers, B, total_probe, total_ctx);
  for (int32_t l = 0; l < n_layers; l += at_once) {
    const int n = std::min(at_once, n_layers - l);
    const float beta = l == 0 ? 0.f : 1.f;
    if (n == 1) {
      QCF_TRY(launch_score(L, B, q[l], probe_off, total_probe, k[l], ctx_off, total_ctx, probe_limit, score, weights[l], beta, ws, st));
    } else {
      const ScoreArgs a = score_args(L, B, q[l], probe_off, total_probe, k[l], ctx_off, total_ctx, probe_limit, score, weights[l], beta);
      QCF_TRY(launch_two_pass(L, a, n, q + l, k + l, weights + l, ws, st));
    }
  }
  return QCF_OK;
}

}  // namespace qcf

// ---- scoring for callers that cannot allocate -----------------------------------------------------
// The scratch of the kernels above (tile partials and per-head column sums, or the probability rows of
// the generic path) lives in a device array that is part of the loaded code object: every GPU the library
// runs on holds its own copy, at its own address, until the process ends.  In host code the array's name is
// only a handle: the device address is asked for once per device (with that device current) and kept, and
// that pointer is what the launchers receive.
namespace {

__device__ __align__(256) unsigned char scratch[QCF_SCORE_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::atomic<void*> g_scratch_ptr[kMaxDevices];

qcf_status scratch_of_current_device(void** out) {
  int dev = 0;
  QCF_TRY(qcf::check_hip(hipGetDevice(&dev), "hipGetDevice"));
  if (dev < 0 || dev >= kMaxDevices) return qcf::fail(QCF_ERR_UNSUPPORTED, "device id %d >= %d", dev, kMaxDevices);
  void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (!p) {
    // (two threads may both ask; they get the same address)
    QCF_TRY(qcf::check_hip(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)"));
    if (!p) return qcf::fail(QCF_ERR_HIP, "hipGetSymbolAddress(scratch) returned a null address");
    g_scratch_ptr[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return QCF_OK;
}

}  // namespace

extern "C" qcf_status qcf_score_static(const qcf_layer_desc* desc, int32_t B, const void* q_probe,
                                       const int64_t* probe_off_dev, int64_t total_probe, const void* k_fused,
                                       const int64_t* ctx_off_dev, int64_t total_ctx,
                                       const int32_t* probe_limit_dev, float* score, void* stream) {
  bool empty = false;
  QCF_TRY(qcf::check_score_args(desc, B, q_probe, probe_off_dev, total_probe, k_fused, ctx_off_dev, total_ctx,
                                probe_limit_dev, score, &empty));
  if (empty) return QCF_OK;
  const size_t need = qcf::scoring::workspace(*desc, B, total_probe, total_ctx);
  if (need > (size_t)QCF_SCORE_STATIC_SCRATCH_BYTES)
    return qcf::fail(QCF_ERR_WORKSPACE_TOO_SMALL,
                     "qcf_score_static: this problem needs %zu bytes of scratch, the built-in buffer has %zu; "
                     "use qcf_score with a caller-supplied workspace",
                     need, (size_t)QCF_SCORE_STATIC_SCRATCH_BYTES);
  void* ws = nullptr;
  QCF_TRY(scratch_of_current_device(&ws));
  return qcf::launch_score(*desc, B, q_probe, probe_off_dev, total_probe, k_fused, ctx_off_dev, total_ctx,
                           probe_limit_dev, score, 1.f, 0.f, ws, (hipStream_t)stream);
}
