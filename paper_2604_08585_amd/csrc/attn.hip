// Step 6: location-aware sparse causal attention (Section 3.2 of the paper): the selected
// rows, given with their absolute positions, attend over the patched fused cache.
//
// bf16 / head_dim 128 and 64 path: flash-style online softmax on 32x32x16 MFMA.  A workgroup owns a
// block of consecutive selected rows times the G query heads of one KV head (128 "rows"), so
// every K/V tile is loaded once per KV head.  Logits are produced transposed (S^T = K Q^T):
// a lane then owns one row and the softmax statistics need no cross-lane traffic beyond one
// exchange between the two lane halves; the probabilities, still in registers, are already
// the B operand of O^T += V^T P^T.  V tiles are transposed on their way into LDS.  Key tiles
// wholly above a wave's highest position are skipped, tiles wholly below its lowest run
// unmasked, only the straddling tiles compare positions.  When the launch has too few row blocks
// to balance the causal triangle over the compute units, a row block's keys are cut into segments
// that run as separate workgroups; each writes a normalised partial output and its log-sum-exp,
// and a second kernel merges them (the usual softmax merge, exact up to rounding).
//
// Heads of 64: the probabilities enter the second product as three bf16 terms that add up to the float, and the partial
// outputs of split row blocks are fp32, so nothing between the operands and the stored result is rounded to bf16 (with two
// terms 3.1 times as many results were not the bf16 nearest to the exact one as with float32 products: 3893 to 1237 of
// 4.4 million; with three 642).  Rows that come out infinite or NaN are computed again in a second sweep over the same
// tiles (see there).
// Bound by the softmax arithmetic between the two products and by the splitting into terms.  615 rows x 32 heads over 4096
// tokens: 1580 us with the generic kernel, 48.0 us here (41.7 with two terms); the whole layer 96.6 us (2074 before).
//
// Generic path (f32, or other shapes): one workgroup per (row, head) or pair of heads, online softmax over
// tiles of 256 or 512 tokens.  Bound by the latency of its loads where rows are few and by their number where they are many.
#include "attn_common.h"

namespace qcf {
using namespace attn;
namespace {

// ------------------------------------------------------------------ generic path

// bfloat16.  A tile of 256 tokens: keys a token to a thread, values four elements of every kSlices-th token to a thread, kBatch
// vectors of either on their way.  kBatch 16: the keys and the first 16 values are requested together, so that a tile waits for
// memory once.  Launches of kManyWgs workgroups to a compute unit hide the waits behind each other and lose by the registers
// (170, heads of 128): kBatch 8, values behind the keys, waves without a token of the last tile pass it over.  The sums and their
// order are the same.  us, 16 and 8: 12 / 4 heads of 128, 300 rows over 512 69 and 61, 77 over 512 22.1 and 23.3; heads of 64
// (130 registers) 614 rows over 4096 356 and 400, 300 over 512 36.3 and 38.0.  (Lanes that share a token, as below, lose here, where a
// token takes 128 or 256 bytes: 300 over 512 60 and 83.)
constexpr int kManyWgs = 5;
template <int D, int kBatch>
__global__ __launch_bounds__(256) void attn_generic(AttnArgs a) {
  typedef bf16_t T;
  constexpr int kQuads = D / 4, kSlices = 256 / kQuads, kVals = 256 / kSlices;
  constexpr bool kTogether = kBatch == 16;
  __shared__ __align__(16) float sq[D];
  __shared__ float sp[256];
  __shared__ __align__(16) float sacc[kSlices * D];
  __shared__ float redm[4], reds[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = blockIdx.x / a.H;
  const int h = blockIdx.x - (int)row * a.H;
  // (everything that does not depend on the request is requested in front of the search for it: one wait instead of three)
  const float q1 = tid < D ? Elem<T>::load(static_cast<const T*>(a.q) + (row * a.H + h) * D + tid) : 0.f;
  const int pos = a.sel_pos[row];
  int64_t ctx0 = a.ctx_off[0], ctx1 = a.ctx_off[1];
  const int b = find_request(a.sel_off, a.B, row);
  if (b >= a.B) return;
  if (b > 0) { ctx0 = a.ctx_off[b]; ctx1 = a.ctx_off[b + 1]; }
  const int64_t c0 = min(max(ctx0, (int64_t)0), a.total_ctx);
  const int64_t c1 = min(max(ctx1, c0), a.total_ctx);
  const int Tn = (int)(c1 - c0);
  const int64_t p0 = a.ctx_pos0 ? a.ctx_pos0[b] : 0;
  const int n_vis = (int)min((int64_t)Tn, max((int64_t)0, (int64_t)pos - p0 + 1));
  const int g = h / a.G;
  const T* kb = static_cast<const T*>(a.k) + (c0 * a.Hkv + g) * D;
  const T* vb = static_cast<const T*>(a.v) + (c0 * a.Hkv + g) * D;
  const int64_t kv_stride = (int64_t)a.Hkv * D;
  if (tid < D) sq[tid] = q1 * rsqrtf((float)D);
  __syncthreads();
  const int quad = tid % kQuads, slice = tid / kQuads;       // values: the slices' sums are added in order at the end
  float m_run = -INFINITY, l_run = 0.f, acc[4] = {0.f, 0.f, 0.f, 0.f};
  for (int j0 = 0; j0 < n_vis; j0 += 256) {
    const int n = min(256, n_vis - j0);
    const T* kr = kb + (int64_t)(j0 + min(tid, n - 1)) * kv_stride;
    const T* vt = vb + (int64_t)j0 * kv_stride + 4 * quad;
    float kf[kBatch][4], vf[kBatch][4];
    auto load_values = [&](int u0) {
#pragma unroll
      for (int u = 0; u < kBatch; ++u) Quad<T>::load(vt + (int64_t)min(slice + (u0 + u) * kSlices, n - 1) * kv_stride, vf[u]);
    };
    float s = 0.f;
    if (kTogether || 64 * __builtin_amdgcn_readfirstlane(wave) < n) {
#pragma unroll
      for (int c = 0; c < kQuads; c += kBatch) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) Quad<T>::load(kr + 4 * (c + u), kf[u]);
        if (kTogether && c + kBatch == kQuads) load_values(0);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
          const float4 w = *reinterpret_cast<const float4*>(sq + 4 * (c + u));
          s += w.x * kf[u][0];
          s += w.y * kf[u][1];
          s += w.z * kf[u][2];
          s += w.w * kf[u][3];
        }
      }
    }
    if (tid >= n) s = -INFINITY;
    float mx = s;
    for (int d = 32; d >= 1; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
    if (lane == 0) redm[wave] = mx;
    __syncthreads();                               // (and the previous tile's probabilities have been read)
    mx = fmaxf(fmaxf(redm[0], redm[1]), fmaxf(redm[2], redm[3]));
    const float m_new = fmaxf(m_run, mx);          // finite: the tile has at least one visible token
    const float p = tid < n ? expf(s - m_new) : 0.f;
    sp[tid] = p;
    float sum = p;
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) reds[wave] = sum;
    __syncthreads();
    sum = (reds[0] + reds[1]) + (reds[2] + reds[3]);
    const float alpha = expf(m_run - m_new);       // 0 on the first tile
    l_run = l_run * alpha + sum;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] *= alpha;
#pragma unroll
    for (int u0 = 0; u0 < kVals; u0 += kBatch) {
      if (slice + u0 * kSlices >= n) break;
      if (!kTogether || u0 > 0) load_values(u0);
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int jj = slice + (u0 + u) * kSlices;
        const float w = sp[jj];
        if (jj < n) {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] += w * vf[u][e];
        }
      }
    }
    m_run = m_new;
  }
  *reinterpret_cast<float4*>(sacc + slice * D + 4 * quad) = make_float4(acc[0], acc[1], acc[2], acc[3]);
  __syncthreads();
  if (tid < D) {
    float o = sacc[tid];
    for (int w = 1; w < kSlices; ++w) o += sacc[w * D + tid];
    Elem<T>::store(static_cast<T*>(a.o) + (row * a.H + h) * D + tid, n_vis > 0 ? o / l_run : 0.f);
  }
  if (tid == 0 && a.lse) a.lse[row * a.H + h] = n_vis > 0 ? m_run + logf(l_run) : -INFINITY;
}

// float32: D / 4 lanes take a token, so that a load brings whole key rows (a token to a thread asked for 64 lines with every load),
// and NH heads of a KV group share a workgroup with its keys and values: two where a group has an even number.  Tiles of 512
// tokens, whose keys are dealt to the waves a load at a time and whose values to the slices, as many loads as the tile has tokens
// for: by 64 tokens to a wave, a short tile was one wave's work.  Bound by latency where rows are few, by the reductions and the
// probabilities' arithmetic where they are many.  us, with a token to a thread and a head to a workgroup, with 64 tokens to a wave, and
// so: 4 / 2 heads of 64, 77 rows over 64 tokens 6.1, 6.4, 4.7, over 512 11.1, 8.0, 7.7, 300 over 2048 67.7, 37.0, 31; 3 heads, 1200
// over 64 14.6, 18.3, 12.0; 32 / 8 heads of 128, one row over 64 5.5, 8.1, 4.8, 300 over 512 209, 98.6, 73.2; 8 heads, 1200 over 64
// 59.6, 71.2, 30.4.  Error against 64 bits 4.3e-7, 2.0e-7, 2.0e-7 (the last two have the same bits).
// Launches of at most kFewWgs workgroups to a compute unit take 512 threads, which halves the chain of waits; more of them hide each
// other's with 256.  The sums and their order are the same.  512 and 256 threads: 4 / 2 heads of 64, 77 rows (154 workgroups) over
// 512 tokens 7.8 and 10.8, 300 (600) over 64, 512 and 2000 7.6 and 6.7, 11.7 and 12.5, 29.7 and 37.0; 3 heads, 200 (600) over 700
// 10.8 and 13.0; 8 requests of 512, 80 rows each (1280) 21.2 and 20.3; 16 / 8 heads, 300 (2400) over 1000 44.8 and 41.5.
constexpr int kFewWgs = 3;
constexpr int kTileF32 = 512;
// n loads, eight on their way at a time; what is left in a batch of eight, four or two
template <typename F>
__device__ __forceinline__ void in_batches(int n, F&& f) {
  int c = 0;
  for (; c + 4 < n; c += 8) f(c, std::integral_constant<int, 8>{});
  if (c + 2 < n) f(c, std::integral_constant<int, 4>{});
  else if (c < n) f(c, std::integral_constant<int, 2>{});
}
template <int D, int NH, int THREADS>
__global__ __launch_bounds__(THREADS) void attn_generic_f32(AttnArgs a) {
  constexpr int kQuads = D / 4, kSlices = kTileF32 / kQuads, kWaves = kTileF32 / 64;     // of a tile
  constexpr int kTurns = kTileF32 / THREADS;                 // a thread has token and slice tid of each part of THREADS tokens
  constexpr int kTokens = 64 / kQuads;                       // of a load of keys
  constexpr int kDeal = THREADS / 64;                        // waves that the groups of tokens are dealt to
  static_assert(kTileF32 / kTokens / kDeal % 8 == 0 && kTileF32 / kSlices % 8 == 0, "a whole tile is whole batches");
  __shared__ float sp[NH][kTileF32], slog[NH][kTileF32];
  __shared__ __align__(16) float sacc[NH][kSlices * D];
  __shared__ float redm[NH][kWaves], reds[NH][kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int per_row = a.H / NH;
  const int64_t row = blockIdx.x / per_row;
  const int h0 = (int)(blockIdx.x - row * per_row) * NH;
  const int quad = tid % kQuads, slice0 = tid / kQuads, token = lane / kQuads;
  // (everything that does not depend on the request is requested in front of the search for it)
  const float* qp = static_cast<const float*>(a.q) + (row * a.H + h0) * D + 4 * quad;
  float q4[NH][4];
#pragma unroll
  for (int i = 0; i < NH; ++i) Quad<float>::load(qp + i * D, q4[i]);
  const int pos = a.sel_pos[row];
  int64_t ctx0 = a.ctx_off[0], ctx1 = a.ctx_off[1];
  const int b = find_request(a.sel_off, a.B, row);
  if (b >= a.B) return;
  if (b > 0) { ctx0 = a.ctx_off[b]; ctx1 = a.ctx_off[b + 1]; }
  const int64_t c0 = min(max(ctx0, (int64_t)0), a.total_ctx);
  const int64_t c1 = min(max(ctx1, c0), a.total_ctx);
  const int Tn = (int)(c1 - c0);
  const int64_t p0 = a.ctx_pos0 ? a.ctx_pos0[b] : 0;
  const int n_vis = (int)min((int64_t)Tn, max((int64_t)0, (int64_t)pos - p0 + 1));
  const int g = h0 / a.G;
  const uint32_t stride = (uint32_t)a.Hkv * D * sizeof(float);        // of a token; a tile's offsets are below 2^28 (1024 heads at most)
  const char* kb = reinterpret_cast<const char*>(static_cast<const float*>(a.k) + (c0 * a.Hkv + g) * D);
  const char* vb = reinterpret_cast<const char*>(static_cast<const float*>(a.v) + (c0 * a.Hkv + g) * D);
  auto load4 = [&](const char* tile, int j, float* f) { Quad<float>::load(reinterpret_cast<const float*>(tile + (j * stride + 16u * quad)), f); };
  const float scale = rsqrtf((float)D);
  float m_run[NH], l_run[NH], acc[kTurns][NH][4];
#pragma unroll
  for (int i = 0; i < NH; ++i) {
    m_run[i] = -INFINITY;
    l_run[i] = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      q4[i][e] *= scale;
#pragma unroll
      for (int t = 0; t < kTurns; ++t) acc[t][i][e] = 0.f;
    }
  }
  for (int j0 = 0; j0 < n_vis; j0 += kTileF32) {
    const int n = min(kTileF32, n_vis - j0);
    const char* kr = kb + (int64_t)j0 * stride;
    const char* vr = vb + (int64_t)j0 * stride;
    // logits: groups of kTokens tokens are dealt to the waves, so that a short tile is all waves' work
    auto logits = [&](int c, auto n_c) {
      constexpr int N = decltype(n_c)::value;
      float kf[N][4];
#pragma unroll
      for (int u = 0; u < N; ++u)
        load4(kr, min(((c + u) * kDeal + wave) * kTokens + token, n - 1), kf[u]);
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int i = 0; i < NH; ++i) {
          float d = q4[i][0] * kf[u][0];
#pragma unroll
          for (int e = 1; e < 4; ++e) d += q4[i][e] * kf[u][e];
          d = kQuads == 16 ? row_sum(d) : half_wave_sum(d);
          if (quad == 0) slog[i][((c + u) * kDeal + wave) * kTokens + token] = d;
        }
    };
    const int groups = ((n + kTokens - 1) / kTokens - wave + kDeal - 1) / kDeal;      // of this wave (none: 0 or less)
    in_batches(groups, logits);
    __syncthreads();
    float s[kTurns][NH];
#pragma unroll
    for (int t = 0; t < kTurns; ++t) {
      const int at = t * THREADS + 64 * wave;                // this wave's 64 tokens
#pragma unroll
      for (int i = 0; i < NH; ++i) {
        s[t][i] = at + lane < n ? slog[i][at + lane] : -INFINITY;
        const float mx = wave_max(s[t][i]);
        if (lane == 0) redm[i][at / 64] = mx;
      }
    }
    __syncthreads();                               // (and the previous tile's probabilities have been read)
    float alpha[NH];
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      float mx = redm[i][0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) mx = fmaxf(mx, redm[i][w]);
      const float m_new = fmaxf(m_run[i], mx);     // finite: the tile has at least one visible token
#pragma unroll
      for (int t = 0; t < kTurns; ++t) {
        const int at = t * THREADS + 64 * wave;
        const float p = at + lane < n ? expf(s[t][i] - m_new) : 0.f;
        sp[i][at + lane] = p;
        const float sum = wave_sum(p);
        if (lane == 0) reds[i][at / 64] = sum;
      }
      alpha[i] = expf(m_run[i] - m_new);           // 0 on the first tile
      m_run[i] = m_new;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NH; ++i) {
      float sum = 0.f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) sum += reds[i][w];
      l_run[i] = l_run[i] * alpha[i] + sum;
#pragma unroll
      for (int t = 0; t < kTurns; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[t][i][e] *= alpha[i];
    }
#pragma unroll
    for (int t = 0; t < kTurns; ++t) {
      const int slice = slice0 + t * (THREADS / kQuads);
      auto values = [&](int u0, auto n_c) {
        constexpr int N = decltype(n_c)::value;
        float vf[N][4];
#pragma unroll
        for (int u = 0; u < N; ++u) load4(vr, min(slice + (u0 + u) * kSlices, n - 1), vf[u]);
#pragma unroll
        for (int u = 0; u < N; ++u) {
          const int jj = slice + (u0 + u) * kSlices;
          if (jj < n) {
#pragma unroll
            for (int i = 0; i < NH; ++i) {
              const float w = sp[i][jj];
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[t][i][e] += w * vf[u][e];
            }
          }
        }
      };
      in_batches((n + kSlices - 1) / kSlices, values);
    }
  }
#pragma unroll
  for (int t = 0; t < kTurns; ++t)
#pragma unroll
    for (int i = 0; i < NH; ++i)
      *reinterpret_cast<float4*>(&sacc[i][(slice0 + t * (THREADS / kQuads)) * D + 4 * quad]) =
          make_float4(acc[t][i][0], acc[t][i][1], acc[t][i][2], acc[t][i][3]);
  __syncthreads();
  if (tid < NH * D) {                              // the slices' sums in order
    const int i = tid / D, d = tid % D;
    float o = sacc[i][d];
    for (int w = 1; w < kSlices; ++w) o += sacc[i][w * D + d];
    float l = l_run[0];
#pragma unroll
    for (int u = 1; u < NH; ++u) l = i == u ? l_run[u] : l;
    static_cast<float*>(a.o)[(row * a.H + h0 + i) * D + d] = n_vis > 0 ? o / l : 0.f;
  }
  if (tid == 0 && a.lse) {
#pragma unroll
    for (int i = 0; i < NH; ++i) a.lse[row * a.H + h0 + i] = n_vis > 0 ? m_run[i] + logf(l_run[i]) : -INFINITY;
  }
}

// ------------------------------------------------------------------ MFMA path (bf16, d = 128 or 64)

// Second and third bf16 term of two probabilities whose first terms are `pk`: a float has 24 significant bits, each term
// takes eight and the differences are exact, so the three terms add up to the float.
__device__ __forceinline__ void split_rest(float p0, float p1, uint32_t pk, uint32_t& second, uint32_t& third) {
  const float r0 = p0 - __uint_as_float(pk << 16), r1 = p1 - __uint_as_float(pk & 0xffff0000u);
  second = cvt_pk_bf16(r0, r1);
  third = cvt_pk_bf16(r0 - __uint_as_float(second << 16), r1 - __uint_as_float(second & 0xffff0000u));
}

__device__ __forceinline__ bool all_finite(const u32x4& v) {       // eight bf16 values: no exponent field is all ones
  uint32_t x = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) x |= (v[w] & 0x7f807f80u) + 0x00800080u;
  return (x & 0x80008000u) == 0u;
}
// Classes of eight bf16 values (as four pairs): `code` gets 1 for +infinity, 128 for -infinity and 16384 for NaN, as bf16,
// and 0 for finite ones (sums over the 64 tokens of a tile keep the classes apart); `fin` the finite values, 0 for the
// others.
__device__ __forceinline__ void split_classes(const u32x4& v, u32x4& fin, u32x4& code) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    uint32_t f = 0, c = 0;
#pragma unroll
    for (int h = 0; h < 32; h += 16) {
      const uint32_t x = (v[w] >> h) & 0xffffu;
      const bool finite = (x & 0x7f80u) != 0x7f80u;
      const uint32_t cls = (x & 0x7fu) ? 0x4680u : (x & 0x8000u) ? 0x4300u : 0x3f80u;
      f |= (finite ? x : 0u) << h;
      c |= (finite ? 0u : cls) << h;
    }
    fin[w] = f;
    code[w] = c;
  }
}

// Tile layouts in LDS (d = 128: rows of 256 bytes = 16 chunks of 16 bytes, no padding):
//   keys:   chunk c of token row r sits in slot c ^ (r % 16), so the 16-byte reads of 16 consecutive
//           rows at one chunk index touch 16 different bank groups;
//   values: chunk c of row r sits in slot c ^ (4 * (r % 4)), so the 8-byte transposing reads of
//           8 consecutive rows x 64 bytes touch every bank exactly twice.
// d = 64: rows of 128 bytes, two to a sweep over the banks, so the slots are c ^ (r / 2 % 8) and c ^ (4 * (r / 2 % 2)).
// F32: partial outputs are float (part_is_f32)
template <int D, bool F32>
__global__ __launch_bounds__(256, AttnTile<D>::WGS) void attn_mfma_kernel(AttnArgs a) {
  using C = AttnTile<D>;
  static_assert(kOrderLds <= C::LDS, "ordered_unit works in the tiles' LDS");
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ int s_vis_max[4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);    // wave-uniform: keeps tile addresses in scalar registers
  const int hf = lane >> 5, l32 = lane & 31;
  const int BR = a.block_rows;
  const uint32_t lds0 = lds_offset_of(smem);

  // consecutive workgroup ids land on different XCDs: give each XCD its own KV heads so that a
  // head's keys and values stay in one L2; later row blocks (longer key ranges) are scheduled first
  // Launches without a plan take the row blocks from the last (longest key range) to the first; one request first the top
  // segments of all of them (seg_major): the segments that a block does not have, and that end at once, then come last and not
  // among the first 256, one to a compute unit.  The block that the bound has too many stays behind them: between them its
  // units, which end at once, fall on the same compute units again and again (16 rows over 16384 tokens: 31.1 us, 26.6 so; heads
  // of 64 37.9, 31.8).  Of several requests the blocks that hold no rows are the last ones and go in front.  The others
  // read the unit list attn_plan_kernel sorted by length, or find their place in it themselves; segments are counted from the top of
  // a block's key range, so a block's remainder segment is the one at the start of the context.
  const int g = (int)(blockIdx.x % a.Hkv);
  const int unit = (int)(blockIdx.x / a.Hkv);
  int seg = unit % a.n_seg_max, blk = a.n_row_blocks - 1 - unit / a.n_seg_max;
  if (a.seg_major > 0) {
    const int rest = unit - a.seg_major * a.n_seg_max;
    seg = rest < 0 ? unit / a.seg_major : rest % a.n_seg_max;
    blk = rest < 0 ? a.seg_major - 1 - unit % a.seg_major : a.seg_major + rest / a.n_seg_max;
  }
  if (a.units) {
    if (unit >= a.units[0]) return;
    const int code = a.units[1 + unit];
    blk = code >> 8;
    seg = code & 255;
  } else if (a.own_order) {
    const int code = ordered_unit(a, unit, smem);
    blk = code >> 8;
    seg = code & 255;
  }
  blk = __builtin_amdgcn_readfirstlane(blk);            // (wave-uniform, which the compiler does not see of the divisions)
  seg = __builtin_amdgcn_readfirstlane(seg);
  int wg = blk;
  int b = 0;
  int64_t s0 = 0, s1 = 0;
  for (; b < a.B; ++b) {
    s0 = min(max(a.sel_off[b], (int64_t)0), a.total_sel);
    s1 = min(max(a.sel_off[b + 1], s0), a.total_sel);
    const int nb = (int)((s1 - s0 + BR - 1) / BR);
    if (wg < nb) break;
    wg -= nb;
  }
  if (b >= a.B) return;
  const int64_t c0 = min(max(a.ctx_off[b], (int64_t)0), a.total_ctx);
  const int64_t c1 = min(max(a.ctx_off[b + 1], c0), a.total_ctx);
  const int T = (int)(c1 - c0);
  const int64_t p0 = a.ctx_pos0 ? a.ctx_pos0[b] : 0;

  // this lane's row
  const int r = wave * 32 + l32;
  const int64_t srow = s0 + (int64_t)wg * BR + r / a.G;
  const int head = g * a.G + r % a.G;
  const bool row_ok = srow < s1;
  int vis = 0;                                  // number of visible tokens of this row
  if (row_ok) vis = (int)min((int64_t)T, max((int64_t)0, (int64_t)a.sel_pos[srow] - p0 + 1));
  int wave_vis_max = vis, wave_vis_min = row_ok ? vis : 0x7fffffff;
#pragma unroll
  for (int d = 16; d >= 1; d >>= 1) {
    wave_vis_max = max(wave_vis_max, __shfl_xor(wave_vis_max, d, 64));
    wave_vis_min = min(wave_vis_min, __shfl_xor(wave_vis_min, d, 64));
  }
  if (lane == 0) s_vis_max[wave] = wave_vis_max;
  __syncthreads();
  const int wg_vis_max = max(max(s_vis_max[0], s_vis_max[1]), max(s_vis_max[2], s_vis_max[3]));
  const int n_tiles = (wg_vis_max + kBKV - 1) / kBKV;
  const bool split = n_tiles > a.seg_tiles;
  if (seg > 0 && seg * a.seg_tiles >= n_tiles) return;      // this block has fewer segments
  const int t_end = n_tiles - seg * a.seg_tiles;
  const int t_begin = max(0, t_end - a.seg_tiles);
  if (n_tiles == 0) {                 // nothing visible to any row of the block
    if (row_ok) {
      bf16_t* op = static_cast<bf16_t*>(a.o) + (srow * a.H + head) * D + D / 2 * hf;
#pragma unroll
      for (int i = 0; i < D / 16; ++i) *reinterpret_cast<u32x4*>(op + 8 * i) = u32x4{0u, 0u, 0u, 0u};
      if (a.lse && hf == 0) a.lse[srow * a.H + head] = -INFINITY;
    }
    return;
  }

  // asynchronous tile loads: instruction i of wave w fills rows 16*i + 4*w .. +3 (1 KB; d = 64: rows
  // 32*i + 8*w .. +7); lane L fills 16 bytes, a slot of its row, with the chunk the swizzle assigns to that slot.
  // Tokens past the end of the context are clamped (their probabilities are zero).
  const bf16_t* kg = static_cast<const bf16_t*>(a.k) + (c0 * a.Hkv + g) * D;
  const bf16_t* vg = static_cast<const bf16_t*>(a.v) + (c0 * a.Hkv + g) * D;
  constexpr int LPR = 64 / C::LROWS;                              // lanes per row
  const int ld_row = C::LROWS * wave + lane / LPR;                // + 4 * LROWS * i (does not change the slots)
  const uint32_t row_bytes = (uint32_t)a.Hkv * C::ROW;            // one token row of the cache
  const uint32_t ld_kchunk = (uint32_t)(k_slot<D>(lane % LPR, ld_row) * 16);
  const uint32_t ld_vchunk = (uint32_t)(v_slot<D>(lane % LPR, ld_row) * 16);
  const uint32_t ld_koff = (uint32_t)ld_row * row_bytes + ld_kchunk;
  const uint32_t ld_voff = (uint32_t)ld_row * row_bytes + ld_vchunk;
  auto aload = [&](const bf16_t* src, uint32_t off0, uint32_t chunk, int t, uint32_t dst) {
    const char* base = reinterpret_cast<const char*>(src) + (int64_t)t * kBKV * row_bytes;
    if (t * kBKV + kBKV <= T) {
#pragma unroll
      for (int i = 0; i < C::NLOAD; ++i)
        load_to_lds_at(base + (size_t)(4 * C::LROWS * i) * row_bytes, off0, dst + i * 4096);
    } else {
#pragma unroll
      for (int i = 0; i < C::NLOAD; ++i) {
        const int row = min(4 * C::LROWS * i + ld_row, T - 1 - t * kBKV);
        load_to_lds_at(base, (uint32_t)row * row_bytes + chunk, dst + i * 4096);
      }
    }
  };
  auto aload_k = [&](int t, int st) { aload(kg, ld_koff, ld_kchunk, t, lds0 + st * C::STAGE + wave * 1024); };
  auto aload_v = [&](int t, int st) { aload(vg, ld_voff, ld_vchunk, t, lds0 + st * C::STAGE + C::TILE + wave * 1024); };
  auto aload2 = [&](int t, int st) { aload_k(t, st); aload_v(t, st); };
  aload2(t_begin, 0);

  // stationary query fragments: qf[ks] = row r, elements 16*ks + 8*hf .. +7
  bf16x8 qf[C::KS];
  {
    const bf16_t* qp = static_cast<const bf16_t*>(a.q) + ((row_ok ? srow : s0) * a.H + head) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks) {
      u32x4 t = *reinterpret_cast<const u32x4*>(qp + 16 * ks);
      if (!row_ok) t = u32x4{0u, 0u, 0u, 0u};
      qf[ks] = __builtin_bit_cast(bf16x8, t);
    }
  }

  // per-lane byte offsets of the fragment reads inside a stage
  uint32_t kofs[C::KS];     // key fragment ks: token row l32 (+32), chunk 2*ks + hf
#pragma unroll
  for (int ks = 0; ks < C::KS; ++ks) kofs[ks] = lds0 + l32 * C::ROW + k_slot<D>(2 * ks + hf, l32) * 16;
  // values: the lane addresses the 8-byte piece (token 4*hf + (lane%16)/4, elements d0 .. d0+3) where
  // block q = 4*((lane/16)%2) + lane%4 of a 32-element slice starts at d0 = 16*(q%2) + 4*(q/2); after the
  // transposing read lane (row i = lane%32) holds four consecutive tokens of element
  // 16*(i/4 % 2) + 4*(i/8) + i%4, which makes MFMA output row 8b + 4h + c element 16h + 4b + c
  uint32_t vofs[C::DT];     // value fragment of output tile dt
  {
    const int vq = 4 * ((lane >> 4) & 1) + (lane & 3);
    const int d0 = 16 * (vq & 1) + 4 * (vq >> 1);
    const int vrow = 4 * hf + ((lane & 15) >> 2);
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
      vofs[dt] = lds0 + C::TILE + vrow * C::ROW + v_slot<D>(4 * dt + d0 / 8, vrow) * 16 + (d0 & 4) * 2;
  }

  floatx16 oacc[C::DT];
#pragma unroll
  for (int i = 0; i < C::DT; ++i) oacc[i] = floatx16{0};
  float m_run = -INFINITY;      // running max of the scaled logits (log2 domain), shared by both lane halves
  float l_run = 0.f;            // this lane's share of the running denominator
  const float k2 = C::K2;

  // logits of one 64-token tile, its softmax, and its share of the output.  The logits are computed one tile ahead
  // (register v of s[0] is token kv0 + 8*(v/4) + 4*hf + v%4 against this lane's row, s[1]: + 32), so that their MFMAs
  // run between the exponentials of the current tile; `stage` and `next` are byte offsets of the ring slots of this
  // tile and of the one behind it.
  auto k_frag = [&](const uint32_t stage, int ks, int h) { return lds_read16(kofs[ks] + (stage + (uint32_t)h * 32 * C::ROW)); };
  auto logits = [&](const uint32_t stage, floatx16 (&s)[2]) {
    s[0] = floatx16{0};
    s[1] = floatx16{0};
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        s[h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k_frag(stage, ks, h)), qf[ks], s[h], 0, 0, 0);
  };
  auto process = [&](const uint32_t stage, const uint32_t next, int kv0, floatx16 (&cur)[2], floatx16 (&nxt)[2]) {
    if (kv0 + kBKV > wave_vis_min) {
#pragma unroll
      for (int v = 0; v < 32; ++v) {
        const int j = kv0 + 32 * (v >> 4) + 8 * ((v & 15) >> 2) + 4 * hf + (v & 3);
        cur[v >> 4][v & 15] = (j < vis) ? cur[v >> 4][v & 15] : -INFINITY;
      }
    }
    u32x4 kf[2][2];                    // key fragments of the next tile, one k-step ahead
    kf[0][0] = k_frag(next, 0, 0);
    kf[0][1] = k_frag(next, 0, 1);
    float mx = cur[0][0];
#pragma unroll
    for (int v = 1; v < 32; ++v) mx = fmaxf(mx, cur[v >> 4][v & 15]);
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    // The reference point of the exponentials only moves when the maximum grows by more than 2^8: until
    // then probabilities up to 256 are accumulated against the old one (the final division by the
    // denominator makes the result independent of the reference point), and the running output is
    // rescaled far less often.
    const float m_cand = fmaxf(m_run, mx * k2);
    const bool bump = m_cand > m_run + kLazyRescale;          // also the first visible tile (m_run = -inf)
    const float m_new = bump ? m_cand : m_run;
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = bump ? __builtin_amdgcn_exp2f(m_run - m_use) : 1.f;
    m_run = m_new;
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int i = 0; i < C::DT; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[i][v] *= alpha;
    }
    // One MFMA of the next tile's logits, then the exponentials of 32 / (2 KS) elements.  P^T fragments: step
    // s = v / 8 uses registers 8*s .. 8*s+7 (tokens 16*s + 8*(e/4) + 4*hf + e%4).
    constexpr int NM = 2 * C::KS, PER = 32 / NM;
    u32x4 pf[4], pr[4], ps[4];
    shortx4 vlo[4], vhi[4];            // value fragments, up to three ahead
    auto v_read = [&](int idx) {
      const int s2 = idx / C::DT, dt2 = idx % C::DT;
      vlo[idx & 3] = lds_read_tr(vofs[dt2] + (stage + (16 * s2) * C::ROW));
      vhi[idx & 3] = lds_read_tr(vofs[dt2] + (stage + (16 * s2 + 8) * C::ROW));
    };
    float sum = 0.f;
    nxt[0] = floatx16{0};
    nxt[1] = floatx16{0};
#pragma unroll
    for (int n = 0; n < NM; ++n) {
      const int ks = n >> 1, h = n & 1;
      __builtin_amdgcn_sched_barrier(0);
      nxt[h] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[ks & 1][h]), qf[ks], nxt[h], 0, 0, 0);
      if (ks + 1 < C::KS) kf[(ks + 1) & 1][h] = k_frag(next, ks + 1, h);
      if (n >= NM - 3) v_read(n - (NM - 3));
#pragma unroll
      for (int v = n * PER; v < (n + 1) * PER; v += 2) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[v >> 4][v & 15], k2, -m_use));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[v >> 4][(v & 15) + 1], k2, -m_use));
        sum += p0;
        sum += p1;
        const uint32_t pk = cvt_pk_bf16(p0, p1);
        pf[v >> 3][(v & 7) >> 1] = pk;
        if constexpr (C::SPLIT_P) {
          uint32_t second, third;
          split_rest(p0, p1, pk, second, third);
          pr[v >> 3][(v & 7) >> 1] = second;
          ps[v >> 3][(v & 7) >> 1] = third;
        }
      }
    }
    l_run = l_run * alpha + sum;
#pragma unroll
    for (int idx = 0; idx < 4 * C::DT; ++idx) {
      const int s = idx / C::DT, dt = idx % C::DT;
      __builtin_amdgcn_sched_barrier(0);
      if (idx + 3 < 4 * C::DT) v_read(idx + 3);
      const shortx8 both = __builtin_shufflevector(vlo[idx & 3], vhi[idx & 3], 0, 1, 2, 3, 4, 5, 6, 7);
      const bf16x8 vf = __builtin_bit_cast(bf16x8, both);
      oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, pf[s]), oacc[dt], 0, 0, 0);
      if (C::SPLIT_P) {
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, pr[s]), oacc[dt], 0, 0, 0);
        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, ps[s]), oacc[dt], 0, 0, 0);
      }
    }
  };

  // Ring of two slots for keys and two for values; while tile t is processed, keys up to t + 2 and values up to
  // t + 1 are on their way (the keys of tile t have been used one tile earlier).
  floatx16 s_a[2], s_b[2];
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();                                    // tile t_begin has landed
  if (t_begin + 1 < t_end) aload_k(t_begin + 1, 1);
  if (t_begin * kBKV < wave_vis_max) logits(0u, s_a);
  for (int t = t_begin; t < t_end; t += 2) {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();                                  // keys of t + 1 and values of t have landed; keys of t are used
    if (t + 2 < t_end) aload_k(t + 2, 0);
    if (t + 1 < t_end) aload_v(t + 1, 1);
    if (t * kBKV < wave_vis_max) process(0u, (uint32_t)C::STAGE, t * kBKV, s_a, s_b);
    if (t + 1 >= t_end) break;
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (t + 3 < t_end) aload_k(t + 3, 1);
    if (t + 2 < t_end) aload_v(t + 2, 0);
    if ((t + 1) * kBKV < wave_vis_max) process((uint32_t)C::STAGE, 0u, (t + 1) * kBKV, s_b, s_a);
  }

  // epilogue: output register v of tile dt is element 32*dt + 16*hf + v of this lane's row
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  const int64_t unit_slot = ((int64_t)blk * a.Hkv + g) * a.n_seg_max + seg, part_row = unit_slot * C::WG_ROWS + r;    // of a split block
  bf16_t* orow = static_cast<bf16_t*>(a.o) + (srow * a.H + head) * D + 16 * hf;
  // x(dt, v): value of this lane's element 32 dt + 16 hf + v; m + log2(z): log2-sum-exp
  auto store_split = [&](auto x, float m, float z) {         // partial result of one key segment; merged by attn_merge_kernel
    const int64_t at = (unit_slot * 4 + wave) * (32 * D);                   // in register order (see attn_merge_kernel)
    if constexpr (F32) {
      float* part = static_cast<float*>(a.part_o) + at;
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<float4*>(part + (4 * dt + q) * 256 + lane * 4) = make_float4(x(dt, 4 * q), x(dt, 4 * q + 1), x(dt, 4 * q + 2), x(dt, 4 * q + 3));
    } else {
      bf16_t* part = static_cast<bf16_t*>(a.part_o) + at;
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int h8 = 0; h8 < 16; h8 += 8)
          *reinterpret_cast<u32x4*>(part + (2 * dt + h8 / 8) * 512 + lane * 8) = mk4(cvt_pk_bf16(x(dt, h8), x(dt, h8 + 1)), cvt_pk_bf16(x(dt, h8 + 2), x(dt, h8 + 3)),
                                                                          cvt_pk_bf16(x(dt, h8 + 4), x(dt, h8 + 5)), cvt_pk_bf16(x(dt, h8 + 6), x(dt, h8 + 7)));
    }
    if (hf == 0) {
      if (C::SPLIT_P) reinterpret_cast<float2*>(a.part_lse)[part_row] = make_float2(m, z);
      else a.part_lse[part_row] = m + log2f(z);
    }
  };
  auto store_whole = [&](auto x, float m, float z) {
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
      for (int h8 = 0; h8 < 16; h8 += 8)
        *reinterpret_cast<u32x4*>(orow + 32 * dt + h8) = mk4(cvt_pk_bf16(x(dt, h8), x(dt, h8 + 1)), cvt_pk_bf16(x(dt, h8 + 2), x(dt, h8 + 3)),
                                                             cvt_pk_bf16(x(dt, h8 + 4), x(dt, h8 + 5)), cvt_pk_bf16(x(dt, h8 + 6), x(dt, h8 + 7)));
    if (a.lse && hf == 0) a.lse[srow * a.H + head] = natural_lse<C::SPLIT_P>(m, log2f(z));
  };
  bool bad = false;                                    // this row is computed again below
  if constexpr (C::SPLIT_P) {
    const bool sees = vis > t_begin * kBKV;
    bad = sees && !(l_tot > 0.f && l_tot < INFINITY);
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
      for (int v = 0; v < 16; ++v) bad |= sees && !(fabsf(oacc[dt][v]) < INFINITY);
    const uint64_t lanes = __ballot(bad);               // (lanes l and l + 32 hold one row)
    bad = ((lanes >> l32) | (lanes >> (l32 + 32))) & 1u;
  }
  {
    auto x = [&](int dt, int v) { return oacc[dt][v] * inv; };
    const float m = l_tot > 0.f ? m_run : -INFINITY, z = l_tot > 0.f ? l_tot : 1.f;
    if (split) {
      if (!bad) store_split(x, m, z);
    } else if (row_ok && !bad) {
      store_whole(x, m, z);
    }
  }
  if constexpr (C::SPLIT_P) {
    if (!__syncthreads_or(bad)) return;
    // Some row came out infinite or NaN: the tiles once more, with the finite values in the product and the classes of the
    // others (of tokens that the row sees) beside it, against a reference point that follows the maximum at once.  So a
    // value that a row does not see leaves no trace, and a visible infinity stays one.  Only the rows in question are
    // stored.  Costs a few times the first sweep (615 rows x 32 heads over 4096 tokens, every value NaN: 132 us, one
    // infinite value 81).
    uint32_t cls[C::DT][16];                             // 1: +infinity seen, 2: -infinity, 4: NaN
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt) {
      oacc[dt] = floatx16{0};
#pragma unroll
      for (int v = 0; v < 16; ++v) cls[dt][v] = 0u;
    }
    m_run = -INFINITY;
    l_run = 0.f;
    aload2(t_begin, 0);
    for (int t = t_begin; t < t_end; ++t) {
      const int slot = (t - t_begin) & 1, kv0 = t * kBKV;
      const uint32_t stage = (uint32_t)(slot * C::STAGE);
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();                                   // tile t has landed, the other slot has been read
      if (t + 1 < t_end) aload2(t + 1, slot ^ 1);
      if (kv0 >= wave_vis_max) continue;                 // (wave-uniform; the barrier is at the top)
      logits(stage, s_a);
      float mx = -INFINITY;
#pragma unroll
      for (int v = 0; v < 32; ++v) {
        const int j = kv0 + 32 * (v >> 4) + 8 * ((v & 15) >> 2) + 4 * hf + (v & 3);
        s_a[v >> 4][v & 15] = (j < vis) ? s_a[v >> 4][v & 15] : -INFINITY;
        mx = fmaxf(mx, s_a[v >> 4][v & 15]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float m_new = fmaxf(m_run, mx);              // (unscaled here, so that the largest logit gives exactly 1)
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_use) * k2);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
      floatx16 n[C::DT];                                 // sums of the class codes of this tile's tokens that a row sees
#pragma unroll
      for (int dt = 0; dt < C::DT; ++dt) n[dt] = floatx16{0};
      bool any_cls = false;
#pragma unroll
      for (int s = 0; s < 4; ++s) {                      // 16 tokens: registers 8 s .. 8 s + 7
        u32x4 pf, pr, ps, seen;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const int v = 8 * s + e, j = kv0 + 16 * s + 8 * (e >> 2) + 4 * hf + (e & 3);
          const float p0 = __builtin_amdgcn_exp2f((s_a[v >> 4][v & 15] - m_use) * k2);
          const float p1 = __builtin_amdgcn_exp2f((s_a[v >> 4][(v & 15) + 1] - m_use) * k2);
          l_run += p0;
          l_run += p1;
          pf[e >> 1] = cvt_pk_bf16(p0, p1);
          uint32_t second, third;
          split_rest(p0, p1, pf[e >> 1], second, third);
          pr[e >> 1] = second;
          ps[e >> 1] = third;
          seen[e >> 1] = (j < vis ? 0x3f80u : 0u) | (j + 1 < vis ? 0x3f800000u : 0u);
        }
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt) {
          const shortx4 lo = lds_read_tr(vofs[dt] + (stage + (16 * s) * C::ROW)),
                        hi = lds_read_tr(vofs[dt] + (stage + (16 * s + 8) * C::ROW));
          u32x4 fin = __builtin_bit_cast(u32x4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          if (__any(!all_finite(fin))) {
            u32x4 code;
            split_classes(fin, fin, code);
            n[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, code), __builtin_bit_cast(bf16x8, seen), n[dt], 0, 0, 0);
            any_cls = true;
          }
          const bf16x8 vf = __builtin_bit_cast(bf16x8, fin);
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, pf), oacc[dt], 0, 0, 0);
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, pr), oacc[dt], 0, 0, 0);
          oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, ps), oacc[dt], 0, 0, 0);
        }
      }
      if (any_cls) {
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) {
            const int c = (int)n[dt][v];
            cls[dt][v] |= ((c & 0x7f) ? 1u : 0u) | ((c & 0x3f80) ? 2u : 0u) | ((c >> 14) ? 4u : 0u);
          }
      }
    }
    if (!bad) return;
    const float l = l_run + __shfl_xor(l_run, 32, 64);
    // no weight at all (every visible logit is -infinity): NaN, unless other segments may have some
    const float den = l != 0.f ? 1.f / l : split ? 0.f : __builtin_nanf("");
    auto x = [&](int dt, int v) {
      const uint32_t c = l > 0.f ? cls[dt][v] : 0u;
      const float w = oacc[dt][v] * den;
      return c == 0u ? w : c == 1u ? INFINITY : c == 2u ? -INFINITY : __builtin_nanf("");
    };
    const float m = l != 0.f ? m_run * k2 : split ? -INFINITY : __builtin_nanf(""), z = l != 0.f ? l : 1.f;
    if (split) store_split(x, m, z);
    else store_whole(x, m, z);
  }
}

// Work list of a split launch of several requests, or of more units than ordered_unit handles: one entry per (row block, key segment) that has tiles, bucket-sorted by
// length (longest first) so that the short remainders fill the tail of the schedule.  The order inside a
// bucket depends on the race for the slots; results do not, because every unit's output location is given
// by its (row block, segment).
constexpr int kPlanBins = 64;
__global__ __launch_bounds__(1024) void attn_plan_kernel(AttnArgs a) {
  __shared__ int s_vis[kPlanMaxBlocks];     // largest visible length of each row block
  __shared__ int s_cnt[kPlanBins + 1];
  __shared__ int s_off[kPlanBins + 1];
  const int tid = threadIdx.x;
  const int BR = a.block_rows;
  for (int i = tid; i < a.n_row_blocks; i += 1024) s_vis[i] = 0;
  for (int i = tid; i <= kPlanBins; i += 1024) s_cnt[i] = 0;
  __syncthreads();
  // every selected row raises the visible length of its block
  for (int64_t sr = tid; sr < a.total_sel; sr += 1024) {
    int blk0 = 0, b = 0;
    int64_t s0 = 0, s1 = 0;
    for (; b < a.B; ++b) {
      s0 = min(max(a.sel_off[b], (int64_t)0), a.total_sel);
      s1 = min(max(a.sel_off[b + 1], s0), a.total_sel);
      if (sr >= s0 && sr < s1) break;
      blk0 += (int)((s1 - s0 + BR - 1) / BR);
    }
    if (b >= a.B) continue;
    const int64_t c0 = min(max(a.ctx_off[b], (int64_t)0), a.total_ctx);
    const int64_t c1 = min(max(a.ctx_off[b + 1], c0), a.total_ctx);
    const int64_t p0 = a.ctx_pos0 ? a.ctx_pos0[b] : 0;
    const int vis = (int)min(c1 - c0, max((int64_t)0, (int64_t)a.sel_pos[sr] - p0 + 1));
    atomicMax(&s_vis[blk0 + (int)((sr - s0) / BR)], vis);
  }
  __syncthreads();
  // pass 0 counts the units of every length bucket, pass 1 places them
  for (int pass = 0; pass < 2; ++pass) {
    for (int blk = tid; blk < a.n_row_blocks; blk += 1024) {
      const int n_tiles = (s_vis[blk] + kBKV - 1) / kBKV;
      if (pass == 0) a.blk_tiles[blk] = n_tiles;
      const int n_seg = max(1, (n_tiles + a.seg_tiles - 1) / a.seg_tiles);   // a block without tiles still writes zeros
      for (int sg = 0; sg < n_seg; ++sg) {
        const int len = min(a.seg_tiles, n_tiles - sg * a.seg_tiles);
        const int bin = kPlanBins - (int)((int64_t)max(len, 0) * kPlanBins / a.seg_tiles);   // 0: whole segments
        if (pass == 0) atomicAdd(&s_cnt[bin], 1);
        else a.units[1 + atomicAdd(&s_off[bin], 1)] = (blk << 8) | sg;
      }
    }
    __syncthreads();
    if (pass == 0) {
      if (tid == 0) {
        int run = 0;
        for (int i = 0; i <= kPlanBins; ++i) { s_off[i] = run; run += s_cnt[i]; }
        a.units[0] = run;
      }
      __syncthreads();
    }
  }
}

// Merge of the partial results of split row blocks: kMergeWgs workgroups per (row block, KV head), one
// thread per 8 output elements.  The partial outputs lie in the order of the registers they came from, 32 rows after the other:
// vector (16 bytes) v of lane l at 64 v + l, for row l % 32 and elements 32 dt + 16 (l / 32) + 8 h .. + 7, v = 2 dt + h in bf16
// and 4 dt + 2 h (+ 1) in float, so that a store or load of a wave is 1 KB.
// out = sum_s w_s O_s with w_s = 2^(lse_s - lse), lse = log2 sum_s 2^lse_s.
// weight * value; an infinite or NaN value keeps its class also where the weight has underflowed to 0 (SPLIT_P)
template <bool SPLIT_P>
__device__ __forceinline__ float weighted(float w, float f) {
  if (SPLIT_P) return fabsf(f) < INFINITY ? w * f : f;
  return w * f;
}
template <int D, int ROWS> constexpr int kMergeWgs = ROWS * (D / 8) / 256;
template <int D, int ROWS, bool F32>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a) {
  typedef typename std::conditional<F32, float, bf16_t>::type part_t;
  const int tid = threadIdx.x;
  const int BR = a.block_rows;
  const int part = (int)(blockIdx.x % kMergeWgs<D, ROWS>);
  const int bh = (int)(blockIdx.x / kMergeWgs<D, ROWS>);
  const int g = bh % a.Hkv;
  const int blk = bh / a.Hkv;
  int n_tiles = a.blk_tiles ? a.blk_tiles[blk] : 0;
  if (a.blk_tiles && n_tiles <= a.seg_tiles) return;      // not split: the main kernel wrote the result
  int wg = blk, b = 0;
  int64_t s0 = 0, s1 = 0;
  for (; b < a.B; ++b) {
    s0 = min(max(a.sel_off[b], (int64_t)0), a.total_sel);
    s1 = min(max(a.sel_off[b + 1], s0), a.total_sel);
    const int nb = (int)((s1 - s0 + BR - 1) / BR);
    if (wg < nb) break;
    wg -= nb;
  }
  if (b >= a.B) return;
  if (!a.blk_tiles) {                               // no plan: the key tiles of this block, as the main kernel counts them
    __shared__ int s_vis[4];
    const int64_t sr = s0 + (int64_t)wg * BR + tid;
    int vis = 0;
    if (tid < BR && sr < s1) {
      const int64_t c0 = min(max(a.ctx_off[b], (int64_t)0), a.total_ctx);
      const int64_t c1 = min(max(a.ctx_off[b + 1], c0), a.total_ctx);
      const int64_t p0 = a.ctx_pos0 ? a.ctx_pos0[b] : 0;
      vis = (int)min(c1 - c0, max((int64_t)0, (int64_t)a.sel_pos[sr] - p0 + 1));
    }
    for (int d = 32; d >= 1; d >>= 1) vis = max(vis, __shfl_xor(vis, d, 64));
    if ((tid & 63) == 0) s_vis[tid >> 6] = vis;
    __syncthreads();
    n_tiles = (max(max(s_vis[0], s_vis[1]), max(s_vis[2], s_vis[3])) + kBKV - 1) / kBKV;
    if (n_tiles <= a.seg_tiles) return;
  }
  const int n_seg = (n_tiles + a.seg_tiles - 1) / a.seg_tiles;
  const int item = part * 256 + tid, w32 = item / (4 * D), v8 = item % (4 * D) / 64, lane = item % 64;
  const int r = 32 * w32 + lane % 32, elem = 32 * (v8 >> 1) + 16 * (lane >> 5) + 8 * (v8 & 1);    // row of the block, first element
  const int64_t srow = s0 + (int64_t)wg * BR + r / a.G;
  const bool row_ok = srow < s1;
  const int head = g * a.G + r % a.G;
  // unit (blk, g, seg) wrote slot ((blk * Hkv + g) * n_seg_max + seg)
  const int64_t slot0 = ((int64_t)blk * a.Hkv + g) * a.n_seg_max;
  constexpr int PL = AttnTile<D>::SPLIT_P ? 2 : 1;   // floats per row
  const float* pl = a.part_lse + (slot0 * ROWS + r) * PL;
  constexpr int VECS = sizeof(part_t) / 2;          // 16-byte vectors of 8 elements
  const part_t* po = static_cast<const part_t*>(a.part_o) + (slot0 * ROWS + 32 * w32) * D + (VECS * v8 * 64 + lane) * Elem<part_t>::kVec;
  // four segments at a time: every load first, then the running maximum, the weights and the weighted sum
  constexpr bool SPLIT_P = AttnTile<D>::SPLIT_P;
  bool nan = false;                                 // (SPLIT_P) the denominator of some segment is NaN
  float mx = -INFINITY, wsum = 0.f;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int sg0 = 0; sg0 < n_seg; sg0 += 4) {
    float l[4], z[4];
    u32x4 raw[4][VECS];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool ok = row_ok && sg0 + u < n_seg;
      l[u] = ok ? pl[(int64_t)(sg0 + u) * ROWS * PL] : -INFINITY;
      z[u] = !SPLIT_P || !ok ? 1.f : pl[(int64_t)(sg0 + u) * ROWS * PL + 1];
#pragma unroll
      for (int w = 0; w < VECS; ++w)
        raw[u][w] = ok ? *reinterpret_cast<const u32x4*>(po + (int64_t)(sg0 + u) * ROWS * D + w * 64 * Elem<part_t>::kVec) : u32x4{0u, 0u, 0u, 0u};
    }
    float mn = mx;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      mn = fmaxf(mn, l[u]);
      nan |= z[u] != z[u];
    }
    if (mn > -INFINITY) {
      const float resc = __builtin_amdgcn_exp2f(mx - mn);        // 0 while nothing was visible so far
      wsum *= resc;
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = weighted<SPLIT_P>(resc, acc[e]);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float w = __builtin_amdgcn_exp2f(l[u] - mn);              // 0 for a segment that saw nothing
        if (SPLIT_P) w *= z[u];
        float f[8];
#pragma unroll
        for (int w = 0; w < VECS; ++w) Vec16<part_t>::unpack(raw[u][w], f + w * Elem<part_t>::kVec);
        wsum += w;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] += weighted<SPLIT_P>(w, f[e]);
      }
      mx = mn;
    }
  }
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] *= inv;
  float lse = wsum > 0.f ? natural_lse<SPLIT_P>(mx, log2f(wsum)) : -INFINITY;
  if constexpr (SPLIT_P) {
    if (row_ok && !nan && wsum == 0.f) {            // no weight although tokens are visible
      const int64_t c0 = min(max(a.ctx_off[b], (int64_t)0), a.total_ctx);
      const int64_t c1 = min(max(a.ctx_off[b + 1], c0), a.total_ctx);
      nan = c1 > c0 && (int64_t)a.sel_pos[srow] >= (a.ctx_pos0 ? a.ctx_pos0[b] : 0);
    }
    if (nan) {
      lse = __builtin_nanf("");
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = lse;
    }
  }
  if (row_ok && a.lse && elem == 0) a.lse[srow * a.H + head] = lse;
  // the workgroup's 32 rows x 64 elements leave by whole lines: chunk c (16 bytes) of row r in slot c ^ (r % 8)
  __shared__ u32x4 s_out[32 * 8];
  s_out[(r & 31) * 8 + ((elem / 8 & 7) ^ (r & 7))] = Vec16<bf16_t>::pack(acc);
  __syncthreads();
  const int r_out = 32 * w32 + tid / 8, ch = tid % 8;
  const int64_t srow_out = s0 + (int64_t)wg * BR + r_out / a.G;
  if (srow_out < s1)
    *reinterpret_cast<u32x4*>(static_cast<bf16_t*>(a.o) + (srow_out * a.H + g * a.G + r_out % a.G) * D + (elem & ~63) + 8 * ch) =
        s_out[tid / 8 * 8 + (ch ^ (r_out & 7))];
}

template <int D, int ROWS, bool F32>
qcf_status run_mfma(const AttnArgs& a, hipStream_t st) {
  const int64_t blocks = (int64_t)a.n_row_blocks * a.Hkv;
  if (a.units) {
    attn_plan_kernel<<<dim3(1), dim3(1024), 0, st>>>(a);
    QCF_TRY_LAUNCH("attn plan");
  }
  if constexpr (ROWS == kWideRows) {
    QCF_TRY(run_attn128(a, blocks * a.n_seg_max, st));
  } else {
    static std::atomic<uint64_t> lds_ok{0};
    QCF_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(&attn_mfma_kernel<D, F32>), AttnTile<D>::LDS, lds_ok));
    attn_mfma_kernel<D, F32><<<dim3((unsigned)(blocks * a.n_seg_max)), dim3(256), AttnTile<D>::LDS, st>>>(a);
    QCF_TRY_LAUNCH("attn");
  }
  if (a.n_seg_max > 1) {
    attn_merge_kernel<D, ROWS, F32><<<dim3((unsigned)(blocks * kMergeWgs<D, ROWS>)), dim3(256), 0, st>>>(a);
    return check_launch("attn merge");
  }
  return QCF_OK;
}

bool use_mfma(const qcf_layer_desc& L) {
  const int G = L.n_q_heads / L.n_kv_heads;
  return L.dtype == QCF_DTYPE_BF16 && (L.head_dim == 128 || L.head_dim == 64) && G <= 128 && 128 % G == 0;
}

}  // namespace

size_t attn_workspace(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx) {
  return use_mfma(L) && total_sel > 0 && total_ctx > 0 ? full_workspace(L, B, total_sel, total_ctx) : 0;
}

size_t attn_workspace_needed(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx) {
  return use_mfma(L) && L.head_dim == 128 && total_sel > 0 && total_ctx > 0 ? least_workspace(L, B, total_sel, total_ctx) : 0;
}

qcf_status launch_attn(const qcf_layer_desc& L, int32_t B, const void* q, const int32_t* sel_pos,
                       const int64_t* sel_off, int64_t total_sel, const void* k, const void* v,
                       const int64_t* ctx_off, int64_t total_ctx, const int32_t* ctx_pos0, void* o,
                       float* lse, void* ws, size_t ws_bytes, hipStream_t st) {
  AttnArgs a;
  a.q = q; a.k = k; a.v = v;
  a.sel_pos = sel_pos; a.sel_off = sel_off; a.ctx_off = ctx_off; a.ctx_pos0 = ctx_pos0;
  a.total_sel = total_sel; a.total_ctx = total_ctx;
  a.B = B; a.H = L.n_q_heads; a.Hkv = L.n_kv_heads; a.G = L.n_q_heads / L.n_kv_heads; a.D = L.head_dim;
  a.o = o; a.lse = lse;
  a.n_row_blocks = 0;
  a.block_rows = 0;
  a.seg_tiles = 0x3fffffff; a.n_seg_max = 1; a.part_o = nullptr; a.part_lse = nullptr; a.units = nullptr; a.blk_tiles = nullptr;
  a.own_order = 0; a.seg_major = 0;
  if (use_mfma(L)) {
    const Division d = divide(L, B, total_sel, total_ctx, ws_bytes);
    Split sp = d.split;
    if (workspace_of(L, d) > ws_bytes) sp = Split{0x3fffffff, 1};      // (d = 64 only: optional)
    const int64_t nb = d.n_row_blocks;
    if (nb * a.Hkv * std::max(sp.n_seg_max, d.rows * 16 / 256) > 0x7fffffff)
      return fail(QCF_ERR_UNSUPPORTED, "attn: grid too large");
    a.block_rows = d.rows / a.G;
    a.n_row_blocks = (int)nb;
    a.seg_tiles = sp.seg_tiles;
    a.n_seg_max = sp.n_seg_max;
    if (sp.n_seg_max > 1) {
      if (B == 1) a.seg_major = (int)nb - 1;
      a.part_o = ws;
      char* w = static_cast<char*>(ws);
      a.part_lse = reinterpret_cast<float*>(w + part_o_bytes(L, d));
      // The plan sorts the units for the compute units to take in turn.  Where all of them start at once their order does
      // not matter, and the launch is saved: 110 rows over 731 tokens 22.3 -> 19.0 us, 40 rows over 8192 30.4 -> 23.5.
      // The workgroups of one request find their places themselves (ordered_unit) up to 512 units, which covers the split
      // launches of a request whose blocks are few enough to need the order.  With the launch that writes the list and
      // without, us: 615 rows x 32 heads over 4096 tokens 45.0 and 40.9, the last 615 positions in the place of spread ones
      // 63.4 and 58.7, heads of 64 49.4 and 45.8; 410 rows over 8192 50.7 and 46.9, 1229 over 8192 116.0 and 110.2.  An
      // order from the host, for rows taken to be spread evenly, was 2 us faster still on such rows and up to 18 % slower
      // than the list on rows gathered in two places.
      if (nb * a.Hkv * sp.n_seg_max <= resident_workgroups(d.rows) || sp.part_f32) {      // (short launches: segments of one length)
      } else if (B == 1 && nb * sp.n_seg_max <= kOrderMax && nb <= kOrderBlocks) {
        a.own_order = 1;
      } else {
        a.units = reinterpret_cast<int32_t*>(w + part_o_bytes(L, d) + part_lse_bytes(L, d));
        a.blk_tiles = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(a.units) + units_bytes(d));
      }
    }
    if (a.D == 64) return run_mfma<64, kNarrowRows, true>(a, st);
    if (d.rows == kWideRows) return run_mfma<128, kWideRows, true>(a, st);
    return part_is_f32(a.D, d.rows, sp) ? run_mfma<128, kNarrowRows, true>(a, st) : run_mfma<128, kNarrowRows, false>(a, st);
  }
  if (total_sel * a.H > 0x7fffffff) return fail(QCF_ERR_UNSUPPORTED, "attn: grid too large");
  if (L.dtype == QCF_DTYPE_BF16) {
    const dim3 grid((unsigned)(total_sel * a.H)), block(256);
    if (a.D == 64) attn_generic<64, 16><<<grid, block, 0, st>>>(a);
    else if (total_sel * a.H >= (int64_t)kManyWgs * compute_unit_count()) attn_generic<128, 8><<<grid, block, 0, st>>>(a);
    else attn_generic<128, 16><<<grid, block, 0, st>>>(a);
  } else {
    const bool pairs = a.G % 2 == 0;
    const int64_t wgs = total_sel * (pairs ? a.H / 2 : a.H);
    const bool few = wgs <= kFewWgs * (int64_t)compute_unit_count();
#define QCF_F32(DIM, NH)                                                                                     \
  if (few) attn_generic_f32<DIM, NH, 512><<<dim3((unsigned)wgs), dim3(512), 0, st>>>(a);                     \
  else attn_generic_f32<DIM, NH, 256><<<dim3((unsigned)wgs), dim3(256), 0, st>>>(a)
    if (a.D == 64) { if (pairs) { QCF_F32(64, 2); } else { QCF_F32(64, 1); } }
    else { if (pairs) { QCF_F32(128, 2); } else { QCF_F32(128, 1); } }
#undef QCF_F32
  }
  return check_launch("attn");
}

}  // namespace qcf
