// Step 3: Top-N selection (Section 3.1 Phase 3 / Section 3.2 token selector of the paper).
//
// One 1024-thread workgroup per request.  Scores map to order-preserving 32-bit keys; an
// MSB-first radix select over the bits in which the keys actually differ finds the N-th
// largest key and how many of its ties to admit; a block-wide prefix scan then compacts the
// admitted indices in index order, so the output is ascending and ties go to the lower index.
// Integer work only: exact and deterministic.
#include "qcf_internal.h"

namespace qcf {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kDigitBits = 9;                 // bits resolved per pass (measured best of 8..11 at 8192 keys)
constexpr int kBins = 1 << kDigitBits;
constexpr int kBinsPerLane = kBins / 64;     // the first wave scans the histogram

__device__ __forceinline__ uint32_t order_key(float s) {
  uint32_t u = __float_as_uint(s);
  if (u == 0x80000000u) u = 0u;      // -0 and +0 are the same score
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ uint64_t wave_incl_scan(uint64_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t lo = __shfl_up((uint32_t)v, d, 64);
    const uint32_t hi = __shfl_up((uint32_t)(v >> 32), d, 64);
    if (lane >= d) v += ((uint64_t)hi << 32) | lo;
  }
  return v;
}

struct SelectLds {
  uint32_t merged[kBins];
  uint64_t wave_tot[kWaves];
  uint32_t red_lo[kWaves], red_hi[kWaves];
  uint32_t digit, k;
};

// One request: T scores, N of them to select (0 < N <= T), written from sel_*[o0] on.
// SEG > 0: each thread keeps up to SEG keys of its contiguous segment of seg keys in registers.
// SEG == 0: keys are re-read from global memory in every pass (any length).
template <int SEG>
__device__ __forceinline__ void select_request(SelectLds& lds, const float* __restrict__ s, int64_t c0, int T, int N, int seg,
                                               int64_t o0, int base_pos, int32_t* __restrict__ sel_idx,
                                               int32_t* __restrict__ sel_row, int32_t* __restrict__ sel_pos) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int j0 = min(T, tid * seg), j1 = min(T, j0 + seg);      // (T is at most 2^30)
  const int cnt = j1 - j0;

  uint32_t keys[SEG > 0 ? SEG : 1];
  if (SEG > 0) {
    // segments start at multiples of four: with an aligned request every whole quad is one load
    if (SEG % 4 == 0 && (reinterpret_cast<uintptr_t>(s) & 15u) == 0) {
      if (cnt == SEG) {
#pragma unroll
        for (int i = 0; i < SEG; i += 4) {
          const float4 v = *reinterpret_cast<const float4*>(s + j0 + i);
          const float q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int c = 0; c < 4 && i + c < SEG; ++c) keys[i + c] = order_key(q[c]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < SEG; i += 4) {
          float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
          if (i + 3 < cnt) v = *reinterpret_cast<const float4*>(s + j0 + i);
          else {
            if (i < cnt) v.x = s[j0 + i];
            if (i + 1 < cnt) v.y = s[j0 + i + 1];
            if (i + 2 < cnt) v.z = s[j0 + i + 2];
          }
          const float q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
          for (int c = 0; c < 4 && i + c < SEG; ++c) keys[i + c] = order_key(q[c]);
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < SEG; ++i) keys[i] = (i < cnt) ? order_key(s[j0 + i]) : 0u;
    }
  }
#define QCF_KEY(i) (SEG > 0 ? keys[i] : order_key(s[j0 + (i)]))
#define QCF_FOR_KEYS(i, ...)                                   \
  if (SEG > 0) {                                               \
    _Pragma("unroll") for (int i = 0; i < SEG; ++i) {          \
      if (i < cnt) { __VA_ARGS__ }                             \
    }                                                          \
  } else {                                                     \
    for (int i = 0; i < cnt; ++i) { __VA_ARGS__ }              \
  }

  uint32_t tau = 0;       // key of the N-th largest score
  uint32_t k = (uint32_t)N;   // how many keys equal to tau are admitted

  if (N < T) {
    // range of the keys
    uint32_t lo = 0xffffffffu, hi = 0u;
    QCF_FOR_KEYS(i, { const uint32_t key = QCF_KEY(i); lo = min(lo, key); hi = max(hi, key); })
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      lo = min(lo, (uint32_t)__shfl_xor((int)lo, d, 64));
      hi = max(hi, (uint32_t)__shfl_xor((int)hi, d, 64));
    }
    if (lane == 0) { lds.red_lo[wave] = lo; lds.red_hi[wave] = hi; }
    for (int i = tid; i < kBins; i += kThreads) lds.merged[i] = 0u;
    __syncthreads();
    lo = lds.red_lo[0]; hi = lds.red_hi[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) { lo = min(lo, lds.red_lo[w]); hi = max(hi, lds.red_hi[w]); }

    const uint32_t diff = lo ^ hi;
    int bits = diff ? 32 - __clz((int)diff) : 0;     // low bits in which keys may differ
    uint32_t prefix = (bits >= 32) ? 0u : (hi >> bits);   // common high part
    while (bits > 0) {
      const int w = min(kDigitBits, bits);
      const int shift = bits - w;
      const uint32_t mask = (1u << w) - 1u;
      // (lds.merged[] was cleared before the loop and is cleared again by wave 0 after each pass)
      QCF_FOR_KEYS(i, {
        const uint32_t key = QCF_KEY(i);
        const uint32_t high = (bits >= 32) ? 0u : (key >> bits);
        if (high == prefix) atomicAdd(&lds.merged[(key >> shift) & mask], 1u);
      })
      __syncthreads();
      if (wave == 0) {
        uint32_t c[kBinsPerLane];
        uint32_t tot = 0;
#pragma unroll
        for (int q = 0; q < kBinsPerLane; ++q) {
          c[q] = lds.merged[kBinsPerLane * lane + q];
          tot += c[q];
          lds.merged[kBinsPerLane * lane + q] = 0u;
        }
        uint32_t suffix = tot;               // sum over lanes >= this one
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t o = __shfl_down(suffix, d, 64);
          if (lane + d < 64) suffix += o;
        }
        uint32_t above = suffix - tot;       // keys with a larger digit than this lane's bins
#pragma unroll
        for (int q = kBinsPerLane - 1; q >= 0; --q) {
          if (above < k && k <= above + c[q]) { lds.digit = kBinsPerLane * lane + q; lds.k = k - above; }
          above += c[q];
        }
      }
      __syncthreads();
      prefix = (prefix << w) | lds.digit;
      k = lds.k;
      bits = shift;
    }
    tau = prefix;
  }

  // compaction in index order
  uint32_t n_gt = 0, n_eq = 0;
  if (N < T) {
    QCF_FOR_KEYS(i, { const uint32_t key = QCF_KEY(i); n_gt += key > tau; n_eq += key == tau; })
  } else {
    n_gt = (uint32_t)cnt;
  }
  const uint64_t mine = ((uint64_t)n_eq << 32) | n_gt;
  const uint64_t incl = wave_incl_scan(mine, lane);
  if (lane == 63) lds.wave_tot[wave] = incl;
  __syncthreads();
  uint64_t before = incl - mine;
  for (int w = 0; w < wave; ++w) before += lds.wave_tot[w];
  uint32_t gt_before = (uint32_t)before, eq_before = (uint32_t)(before >> 32);
  const int64_t out0 = o0;
#define QCF_EMIT(j, pos)                                            \
  {                                                                 \
    if (sel_idx) sel_idx[out0 + (pos)] = (j);                       \
    if (sel_row) sel_row[out0 + (pos)] = (int32_t)(c0 + (j));       \
    if (sel_pos) sel_pos[out0 + (pos)] = base_pos + (j);            \
  }
  if (N < T) {
    QCF_FOR_KEYS(i, {
      const uint32_t key = QCF_KEY(i);
      const bool gt = key > tau, eq = key == tau;
      const uint32_t pos = gt_before + min(eq_before, k);
      if ((gt || (eq && eq_before < k)) && pos < (uint32_t)N) QCF_EMIT(j0 + i, pos)
      gt_before += gt;
      eq_before += eq;
    })
  } else {
    for (int i = 0; i < cnt; ++i) QCF_EMIT(j0 + i, gt_before + i)
  }
#undef QCF_EMIT
#undef QCF_KEY
#undef QCF_FOR_KEYS
}

// Keys per thread follow the length of each request: a batch of requests whose total exceeds what registers hold does not
// re-read every key in every pass (sixteen requests of 2K-16K tokens: 56 -> 16 us).  MAX: the most keys per thread that
// registers are kept for (they are allocated for the kernel as a whole); 0: and any longer request.
template <int MAX>
__global__ __launch_bounds__(kThreads) void select_kernel(
    const float* __restrict__ score, const int64_t* __restrict__ ctx_off, int64_t total_ctx,
    const int64_t* __restrict__ sel_off, int64_t total_sel, const int32_t* __restrict__ ctx_pos0,
    int32_t* __restrict__ sel_idx, int32_t* __restrict__ sel_row, int32_t* __restrict__ sel_pos) {
  __shared__ SelectLds lds;
  const int b = blockIdx.x;
  int64_t c0 = ctx_off[b], c1 = ctx_off[b + 1];
  c0 = min(max(c0, (int64_t)0), total_ctx);
  c1 = min(max(c1, c0), total_ctx);
  int64_t o0 = sel_off[b], o1 = sel_off[b + 1];
  o0 = min(max(o0, (int64_t)0), total_sel);
  o1 = min(max(o1, o0), total_sel);
  const int T = (int)(c1 - c0);
  const int N = (int)min((int64_t)T, o1 - o0);
  if (N <= 0) return;
  const float* s = score + c0;
  const int base_pos = ctx_pos0 ? ctx_pos0[b] : 0;
  int seg = (T + kThreads - 1) / kThreads;
  if (seg > 1) seg = (seg + 3) & ~3;
#define QCF_SELECT(SEG) select_request<SEG>(lds, s, c0, T, N, seg, o0, base_pos, sel_idx, sel_row, sel_pos)
  if constexpr (MAX > 0 && MAX <= 8) {
    if (seg <= MAX) QCF_SELECT(MAX);     // (always so: a request is never longer than the total)
  } else {
    if (seg <= 1) QCF_SELECT(1);
    else if (seg <= 4) QCF_SELECT(4);
    else if (seg <= 8) QCF_SELECT(8);
    else if (seg <= 16) QCF_SELECT(16);
    else if (seg <= 32) QCF_SELECT(32);
    else if constexpr (MAX == 0) QCF_SELECT(0);
  }
#undef QCF_SELECT
}

// Offline anchors: Top-N of a chunk, then its key and value rows, by the workgroup that selected them.  Bound by latency: the
// offsets of up to kAnchorChunks chunks travel as kernel arguments (3.6 of the 4 KB a launch can have), so that no copy to
// the device stands in front of the first kernel and no launch between the selection and the gather.  Whole extraction,
// us, with four operations on the stream and now: 64 chunks of 512, 26 rows each, 46 and 27; 4 chunks of 64 40 and 27.
constexpr int kAnchorChunks = 448;
struct AnchorChunks {
  int32_t ctx[kAnchorChunks + 1], sel[kAnchorChunks + 1];        // inside the totals (at most 2^30 rows)
};

template <int MAX>
__global__ __launch_bounds__(kThreads) void select_gather_kernel(const float* __restrict__ score, AnchorChunks ch,
                                                                 const u32x4* __restrict__ k, const u32x4* __restrict__ v,
                                                                 int vec_per_row, int32_t* rows, u32x4* __restrict__ k_out,
                                                                 u32x4* __restrict__ v_out) {
  __shared__ SelectLds lds;
  const int b = blockIdx.x, tid = threadIdx.x;
  const int64_t c0 = ch.ctx[b], o0 = ch.sel[b];
  const int T = ch.ctx[b + 1] - ch.ctx[b];
  const int N = min(T, ch.sel[b + 1] - ch.sel[b]);
  if (N <= 0) return;
  int seg = (T + kThreads - 1) / kThreads;
  if (seg > 1) seg = (seg + 3) & ~3;
  select_request<MAX>(lds, score + c0, c0, T, N, seg, o0, 0, nullptr, rows, nullptr);
  if (!k_out) return;                                            // (rows only: the gather is a launch of its own)
  __syncthreads();                                               // this workgroup's rows are written
  const int64_t out = o0 * vec_per_row;
  const int items = N * vec_per_row;                             // (at most kGatherVecs)
  for (int i0 = tid; i0 < items; i0 += 4 * kThreads) {
    u32x4 kk[4], vv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = min(i0 + u * kThreads, items - 1), m = i / vec_per_row;
      const int64_t src = (int64_t)rows[o0 + m] * vec_per_row + (i - m * vec_per_row);
      kk[u] = k[src];
      vv[u] = v[src];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = i0 + u * kThreads;
      if (i < items) { k_out[out + i] = kk[u]; v_out[out + i] = vv[u]; }
    }
  }
}

}  // namespace

size_t select_workspace(int32_t, int64_t) { return 0; }

qcf_status launch_select(int32_t B, const float* score, const int64_t* ctx_off, int64_t total_ctx,
                         const int64_t* sel_off, int64_t total_sel, const int32_t* ctx_pos0,
                         int32_t* sel_idx, int32_t* sel_row, int32_t* sel_pos, void*, hipStream_t st) {
  const dim3 grid((unsigned)B), block(kThreads);
#define QCF_LAUNCH(MAX) \
  select_kernel<MAX><<<grid, block, 0, st>>>(score, ctx_off, total_ctx, sel_off, total_sel, ctx_pos0, sel_idx, sel_row, sel_pos)
  // A request is never longer than total_ctx.  Up to eight keys per thread the instance of the total serves every request
  // (8192 tokens: 11.1 us, with the choice by length inside one kernel 11.5).
  if (total_ctx <= kThreads) QCF_LAUNCH(1);
  else if (total_ctx <= 4 * kThreads) QCF_LAUNCH(4);
  else if (total_ctx <= 8 * kThreads) QCF_LAUNCH(8);
  else if (total_ctx <= 32 * kThreads) QCF_LAUNCH(32);
  else QCF_LAUNCH(0);
#undef QCF_LAUNCH
  return check_launch("select");
}

// A workgroup copies what its chunk selected up to this many 16-byte vectors of keys (64 rows of 8 heads of 128); with more
// the copy is a launch over all of them (64 chunks of 1024, 128 rows each: 56 us by the workgroups, 44 with the launch; 64
// rows each: 43 both ways).
constexpr int64_t kGatherVecs = 8192;

qcf_status launch_select_gather(const qcf_layer_desc& L, const float* score, int32_t n_chunks, const int64_t* ctx_off,
                                const int64_t* sel_off, const void* k, const void* v, int32_t* rows, void* k_out, void* v_out,
                                hipStream_t st) {
  const int vec_per_row = L.n_kv_heads * L.head_dim * elem_size(L.dtype) / 16;
  const int64_t total_ctx = ctx_off[n_chunks], total_sel = sel_off[n_chunks];
  auto ctx = [&](int32_t c) { return std::min(std::max(ctx_off[c], (int64_t)0), total_ctx); };
  auto sel = [&](int32_t c) { return std::min(std::max(sel_off[c], (int64_t)0), total_sel); };
  int64_t longest = 0, most = 0;
  for (int32_t c = 0; c < n_chunks; ++c) {
    longest = std::max(longest, ctx(c + 1) - ctx(c));
    most = std::max(most, std::min(ctx(c + 1) - ctx(c), sel(c + 1) - sel(c)));
  }
  const bool gather = most * vec_per_row <= kGatherVecs;
  for (int32_t first = 0; first < n_chunks; first += kAnchorChunks) {
    const int n = std::min(kAnchorChunks, n_chunks - first);
    AnchorChunks ch;
    for (int i = 0; i <= n; ++i) {
      ch.ctx[i] = (int32_t)ctx(first + i);
      ch.sel[i] = (int32_t)sel(first + i);
    }
#define QCF_LAUNCH(MAX)                                                                              \
  select_gather_kernel<MAX><<<dim3((unsigned)n), dim3(kThreads), 0, st>>>(                           \
      score, ch, static_cast<const u32x4*>(k), static_cast<const u32x4*>(v), vec_per_row, rows,      \
      gather ? static_cast<u32x4*>(k_out) : nullptr, static_cast<u32x4*>(v_out))
    if (longest <= kThreads) QCF_LAUNCH(1);
    else if (longest <= 8 * kThreads) QCF_LAUNCH(8);
    else if (longest <= 32 * kThreads) QCF_LAUNCH(32);
    else QCF_LAUNCH(0);
#undef QCF_LAUNCH
    QCF_TRY_LAUNCH("anchor select");
  }
  return gather ? QCF_OK : launch_gather(L, k, v, rows, total_sel, total_ctx, k_out, v_out, st);
}

}  // namespace qcf
