// Step 3: Top-N selection (Section 3.1 Phase 3 / Section 3.2 token selector of the paper).
//
// One 1024-thread workgroup per request.  Scores map to order-preserving 32-bit keys; a histogram over the range that the
// keys span finds the bin of the N-th largest, the few keys of that bin are ranked against each other (or, where they are
// many, split by a histogram over their own range), and a block-wide prefix count then compacts the admitted indices in index
// order, so the output is ascending and ties go to the lower index.  Integer work only: exact and deterministic.
// Bound by the chain of barriers and latencies (an empty selection takes 1.8 us) and, from about 8192 keys, by the vector
// instructions of one compute unit.  One launch of many, 15 % of T keys selected, us, with a radix select of 9 bits to a pass
// over all keys, contiguous keys per thread and outputs stored one by one, and now: 731 keys 5.9 and 3.8, 4096 8.5 and 5.1,
// 8192 10.5 and 6.5, 32768 25.8 and 14.7, 40000 137 and 26.9; 18 requests of 2000 to 16000 21.0 and 12.0.
#include <type_traits>

#include "qcf_internal.h"
#include "score_layout.h"

namespace qcf {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kDigitBits = 10;               // bits resolved per histogram (8192 keys: 9 bits 6.8 us, 10 6.4)
constexpr int kBins = 1 << kDigitBits;
static_assert(kBins == kThreads && kWaves == 16, "a thread has one bin, a row of lanes the waves' sums");
constexpr int kRanked = 128;                 // keys of one bin that are ranked against each other, and not split further (64 and 256 alike)
constexpr int kListed = kThreads;            // keys of one bin that are listed, one to a thread, and not looked for again
constexpr int kStage = 8192;                 // outputs that leave together

__device__ __forceinline__ uint32_t order_key(float s) {
  uint32_t u = __float_as_uint(s);
  if (u == 0x80000000u) u = 0u;      // -0 and +0 are the same score
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}
// Least and largest value of the 16 lanes of a row (row_ror).
__device__ __forceinline__ uint32_t row_min(uint32_t x) {
  x = min(x, dpp<0x128>(x)); x = min(x, dpp<0x124>(x)); x = min(x, dpp<0x122>(x));
  return min(x, dpp<0x121>(x));
}
__device__ __forceinline__ uint32_t row_max(uint32_t x) {
  x = max(x, dpp<0x128>(x)); x = max(x, dpp<0x124>(x)); x = max(x, dpp<0x122>(x));
  return max(x, dpp<0x121>(x));
}
__device__ __forceinline__ uint32_t from_lane(uint32_t x, int lane) { return (uint32_t)__builtin_amdgcn_readlane((int)x, lane); }
// Inclusive sum over the lanes of a wave: within rows (row_shr), then across them (row_bcast).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x) {
  x += dpp<0x111>(x); x += dpp<0x112>(x); x += dpp<0x114>(x); x += dpp<0x118>(x);
  x += dpp<0x142, 0xa>(x);
  return x + dpp<0x143, 0xc>(x);
}
// Sum of x over the first i + 1 of 16 lanes, where every row of the wave has the same sixteen values.
__device__ __forceinline__ uint32_t row_incl_scan_at(uint32_t x, int i) {
  x += dpp<0x111>(x); x += dpp<0x112>(x); x += dpp<0x114>(x); x += dpp<0x118>(x);
  return from_lane(x, i);
}
__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {    // set bits of the lanes before this one
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

struct SelectLds {
  uint32_t merged[kBins];
  uint32_t listed[kListed];
  uint32_t wave_sum[kWaves], wave_gt[kWaves], wave_eq[kWaves];
  uint32_t red_lo[kWaves], red_hi[kWaves];
  uint32_t digit, k, count, n_listed;
  int32_t list[kStage];              // the selected indices of the last window, from which they leave
};

// One request: T scores, N of them to select (0 < N <= T), written from sel_*[o0] on.  Wave w has the keys from w * 64 * seg
// on, in rows of 64 (seg == 1) or 256 (seg a multiple of four: 4 to a lane), so that loads are whole lines.
// SEG > 0: each thread keeps up to SEG keys in registers.  SEG == 0: keys are re-read in every pass (any length).
// WHOLE: no wave lacks a row (or there is one key to a thread).  Otherwise rows that are not there are passed over: taken for keys
// of 0 they cost time and, where the keys' range reaches down to 0 (scores of both signs), crowd one bin: 20000 keys of a normal
// distribution 27.0 us, 14.0 so, 1300 9.0 and 6.8; all equal 13.5 and 10.0.  (The branches cost 2 to 4 % where no row is missing.)
template <int SEG, bool WHOLE>
__device__ __forceinline__ void select_rows(SelectLds& lds, const float* __restrict__ s, int64_t c0, int T, int N, int seg,
                                               int64_t o0, int base_pos, int32_t* __restrict__ sel_idx,
                                               int32_t* __restrict__ sel_row, int32_t* __restrict__ sel_pos) {
  constexpr int C = SEG == 1 ? 1 : 4, kRows = SEG / C;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto emit = [&](int pos, int j) {
    if (sel_idx) sel_idx[o0 + pos] = j;
    if (sel_row) sel_row[o0 + pos] = (int32_t)(c0 + j);
    if (sel_pos) sel_pos[o0 + pos] = base_pos + j;
  };
  if (N == T) {
    for (int j = tid; j < T; j += kThreads) emit(j, j);
    return;
  }
  seg = max(seg, C);
  const int first = wave * 64 * seg + lane * C;                  // this lane's first key (T is at most 2^30)
  const int left = min(T, (wave + 1) * 64 * seg) - first;        // key c of row q exists: 64 * C * q + c < left
  const int rows = min(seg / C, (max(0, T - wave * 64 * seg) + 64 * C - 1) / (64 * C));
  const int rows_full = min(seg / C, max(0, T - wave * 64 * seg) / (64 * C));
  const bool quads = C == 4 && (reinterpret_cast<uintptr_t>(s) & 15u) == 0;
  auto load_row = [&](int q, uint32_t (&bits)[C]) {              // (branches of whole waves: the loads stay in flight)
    const int j = first + 64 * C * q;
    if (q < rows_full && quads) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(s + j);
#pragma unroll
      for (int c = 0; c < C; ++c) bits[c] = v[c];
    } else if (q < rows) {
#pragma unroll
      for (int c = 0; c < C; ++c) bits[c] = __float_as_uint(s[min(j + c, T - 1)]);
    } else {
#pragma unroll
      for (int c = 0; c < C; ++c) bits[c] = 0u;
    }
  };
  // A key of the last row that is not there is 0, what no score but one NaN maps to, and so never among the N < T largest unless
  // that NaN is.
  const bool full = rows_full == (WHOLE && SEG > 0 ? kRows : rows);      // (of the whole wave)
  uint32_t keys[SEG > 0 ? kRows : 1][C];
  uint32_t lo = 0xffffffffu, hi = 0u;                            // range of the keys
  auto order_row = [&](int q, uint32_t (&key)[C]) {
#pragma unroll
    for (int c = 0; c < C; ++c) key[c] = order_key(__uint_as_float(key[c]));
    if (!full) {
#pragma unroll
      for (int c = 0; c < C; ++c) key[c] = 64 * C * q + c < left ? key[c] : 0u;
    }
  };
  auto range_row = [&](int q, const uint32_t (&key)[C]) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      lo = full || 64 * C * q + c < left ? min(lo, key[c]) : lo;
      hi = max(hi, key[c]);
    }
  };
  if constexpr (SEG > 0) {
#pragma unroll
    for (int q = 0; q < kRows; ++q) load_row(q, keys[q]);
    if (full) {
#pragma unroll
      for (int q = 0; q < kRows; ++q)
        if (WHOLE || q < rows) { order_row(q, keys[q]); range_row(q, keys[q]); }
    } else {
#pragma unroll
      for (int q = 0; q < kRows; ++q)
        if (WHOLE || q < rows) { order_row(q, keys[q]); range_row(q, keys[q]); }
    }
  }
  // f(q, key[C]), row by row
  auto walk = [&](auto&& f) {
    if constexpr (SEG > 0) {
#pragma unroll
      for (int q = 0; q < kRows; ++q)
        if (WHOLE || q < rows) f(q, keys[q]);
    } else {
      for (int q = 0; q < rows; ++q) {
        load_row(q, keys[0]);
        order_row(q, keys[0]);
        f(q, keys[0]);
      }
    }
  };
  if constexpr (SEG == 0) walk(range_row);

  lo = row_min(lo);
  hi = row_max(hi);
  lo = min(min(from_lane(lo, 0), from_lane(lo, 16)), min(from_lane(lo, 32), from_lane(lo, 48)));   // (by all lanes: the rows'
  hi = max(max(from_lane(hi, 0), from_lane(hi, 16)), max(from_lane(hi, 32), from_lane(hi, 48)));   // values are there)
  if (lane == 0) { lds.red_lo[wave] = lo; lds.red_hi[wave] = hi; }
  lds.merged[tid] = 0u;
  if (tid == 0) lds.n_listed = 0u;
  __syncthreads();
  lo = __builtin_amdgcn_readfirstlane(row_min(lds.red_lo[lane & 15]));
  hi = __builtin_amdgcn_readfirstlane(row_max(lds.red_hi[lane & 15]));

  // The N-th largest key is top - d for a d of fewer than bits bits: one of count keys, the k-th largest of them.
  uint32_t top = hi, k = (uint32_t)N, tau = hi;
  int bits = hi > lo ? 32 - __clz((int)(hi - lo)) : 0;
  bool listed = SEG == 1;                    // one key to a thread, ones of them (otherwise keys that are not there count too)
  uint32_t one = SEG == 1 ? keys[0][0] : 0u;
  int ones = T;
  uint32_t count = SEG == 1 ? (uint32_t)T : (uint32_t)max(T, kListed + 1);
  while (bits > 0) {
    // (no key is more than 2^bits below the first top, so that top - key of a key above top has a bit above)
    auto in_bin = [&](uint32_t key) { return bits >= 32 || (top - key) >> bits == 0u; };
    if (count <= (uint32_t)(listed ? kRanked : kListed)) {
      auto list = [&](uint32_t key) {
        if (in_bin(key)) {
          const uint32_t at = atomicAdd(&lds.n_listed, 1u);
          if (at < (uint32_t)kListed) lds.listed[at] = key;
        }
      };
      if (listed) {
        if (tid < ones) list(one);
      } else walk([&](int, const uint32_t (&key)[C]) {
#pragma unroll
        for (int c = 0; c < C; ++c) list(key[c]);
      });
      __syncthreads();
      ones = (int)count;
      one = tid < ones ? lds.listed[tid] : 0u;
      listed = true;
      if (count <= (uint32_t)kRanked) {
        if (tid < ones) {
          uint32_t gt = 0, eq = 0;
#pragma unroll 8
          for (int i = 0; i < ones; ++i) {
            const uint32_t o = lds.listed[i];
            gt += o > one;
            eq += o == one;
          }
          if (gt < k && k <= gt + eq) { lds.digit = one; lds.k = k - gt; }     // (the same by all that are equal)
        }
        __syncthreads();
        tau = lds.digit;
        k = lds.k;
        break;
      }
    }
    const int w = min(kDigitBits, bits), shift = bits - w;
    auto add = [&](uint32_t key) {
      const uint32_t bin = (top - key) >> shift;
      if (bin >> w == 0u) atomicAdd(&lds.merged[bin], 1u);
    };
    if (listed) {
      if (tid < ones) add(one);
    } else walk([&](int, const uint32_t (&key)[C]) {
#pragma unroll
      for (int c = 0; c < C; ++c) add(key[c]);
    });
    __syncthreads();
    const uint32_t here = lds.merged[tid], incl = wave_incl_scan(here);
    if (lane == 63) lds.wave_sum[wave] = incl;
    __syncthreads();
    const uint32_t before = row_incl_scan_at(lds.wave_sum[lane & 15], wave) - from_lane(incl, 63) + incl - here;   // larger keys
    if (before < k && k <= before + here) { lds.digit = (uint32_t)tid; lds.k = k - before; lds.count = here; }
    lds.merged[tid] = 0u;
    if (tid == 0) lds.n_listed = 0u;
    __syncthreads();
    top -= lds.digit << shift;
    k = lds.k;
    count = lds.count;
    bits = shift;
    tau = top;
  }
  tau = __builtin_amdgcn_readfirstlane(tau);             // key of the N-th largest score; of those equal to it k are admitted
  k = __builtin_amdgcn_readfirstlane(k);

  // Compaction in index order: the waves' counts, then ballots within a wave.  Where every tie is admitted, as nearly always,
  // the keys from tau on; otherwise the larger ones and the first k of the equal ones.
  uint32_t n_ge = 0;
  walk([&](int, const uint32_t (&key)[C]) {
#pragma unroll
    for (int c = 0; c < C; ++c) n_ge += (uint32_t)__popcll(__ballot(key[c] >= tau));
  });
  if (lane == 0) lds.wave_gt[wave] = n_ge;
  __syncthreads();
  uint32_t gt0 = row_incl_scan_at(lds.wave_gt[lane & 15], wave) - n_ge, eq0 = 0;
  const bool ties = row_incl_scan_at(lds.wave_gt[lane & 15], kWaves - 1) != (uint32_t)N;
  if (ties) {
    uint32_t n_gt = 0, n_eq = 0;
    walk([&](int q, const uint32_t (&key)[C]) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        n_gt += (uint32_t)__popcll(__ballot(key[c] > tau));
        n_eq += (uint32_t)__popcll(__ballot(key[c] == tau && 64 * C * q + c < left));
      }
    });
    __syncthreads();
    if (lane == 0) { lds.wave_gt[wave] = n_gt; lds.wave_eq[wave] = n_eq; }
    __syncthreads();
    gt0 = row_incl_scan_at(lds.wave_gt[lane & 15], wave) - n_gt;
    eq0 = row_incl_scan_at(lds.wave_eq[lane & 15], wave) - n_eq;
  }
  // place(position, key) for every admitted key, positions counted from w0
  auto compact = [&](int w0, auto&& place) {
    uint32_t gt_run = gt0 - (uint32_t)w0, eq_run = eq0, tau_now = tau;
    asm volatile("" : "+s"(tau_now));                            // (compared anew: the masks of the counts are not kept)
    if (!ties) {
      walk([&](int q, const uint32_t (&key)[C]) {
        uint32_t pos = gt_run;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const uint64_t ge = __ballot(key[c] >= tau_now);
          pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(ge >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ge, pos));
          gt_run += (uint32_t)__popcll(ge);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const bool ge = key[c] >= tau_now;
          if (ge) place(pos, first + 64 * C * q + c);
          pos += ge;
        }
      });
    } else {
      int left_now = left;
      asm volatile("" : "+v"(left_now));
      walk([&](int q, const uint32_t (&key)[C]) {
        uint32_t gt = gt_run, eq = eq_run;
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const uint64_t bg = __ballot(key[c] > tau_now), be = __ballot(key[c] == tau_now && 64 * C * q + c < left_now);
          gt += lanes_below(bg);
          eq += lanes_below(be);
          gt_run += (uint32_t)__popcll(bg);
          eq_run += (uint32_t)__popcll(be);
        }
#pragma unroll
        for (int c = 0; c < C; ++c) {
          const bool is_gt = key[c] > tau_now, is_eq = key[c] == tau_now && 64 * C * q + c < left_now;
          if (is_gt || (is_eq && eq < k)) place(gt + min(eq, k), first + 64 * C * q + c);
          gt += is_gt;
          eq += is_eq;
        }
      });
    }
  };
  // More outputs than one window holds: keys in registers are walked again for each (32768 keys, all but 768 selected, 23.9 us),
  // keys that would be read again leave one by one.  A million keys, half of them selected, us: 9850 with 64 windows, 905 so;
  // 157286 selected 3380 and 730; 65536 keys, 19660 selected 56 and 46.
  if constexpr (SEG == 0) {
    if (N > kStage) {
      compact(0, [&](uint32_t pos, int j) {
        if (pos < (uint32_t)N) emit((int)pos, j);
      });
      return;
    }
  }
  for (int w0 = 0; w0 < N; w0 += kStage) {
    compact(w0, [&](uint32_t pos, int j) {
      if (pos < (uint32_t)kStage) lds.list[pos] = j;
    });
    __syncthreads();
    const int n = min(N - w0, kStage);
    for (int i = tid; i < n; i += kThreads) emit(w0 + i, lds.list[i]);
    if (w0 + kStage < N) __syncthreads();
  }
}

template <int SEG>
__device__ __forceinline__ void select_request(SelectLds& lds, const float* __restrict__ s, int64_t c0, int T, int N, int seg,
                                               int64_t o0, int base_pos, int32_t* __restrict__ sel_idx,
                                               int32_t* __restrict__ sel_row, int32_t* __restrict__ sel_pos) {
  if constexpr (SEG == 1)
    select_rows<1, true>(lds, s, c0, T, N, seg, o0, base_pos, sel_idx, sel_row, sel_pos);
  else if (SEG > 0 && seg == SEG && T > SEG * kThreads - 256)
    select_rows<SEG, true>(lds, s, c0, T, N, seg, o0, base_pos, sel_idx, sel_row, sel_pos);
  else
    select_rows<SEG, false>(lds, s, c0, T, N, seg, o0, base_pos, sel_idx, sel_row, sel_pos);
}

// Keys per thread follow the length of each request: a batch of requests whose total exceeds what registers hold does not
// re-read every key in every pass (sixteen requests of 2K-16K tokens, 15 % selected: 23.2 us so, 12.0 now).  MAX: the most keys per thread that
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

// Selection of one request whose scores its workgroup adds up first, in the order of the scoring's own kernels and with their bits,
// so that no launch of a few workgroups stands between the two.  Probability rows: bound by the latency of their loads, up to 48 of a thread
// on their way; shares that a thread does not have and rows that a share does not have are left out, at the sizes below (with
// room for four shares of twelve rows each, always: whole layers of f32, 4 heads, 8 probe rows over 64 tokens 24.6 us, so 21.5, 96 over
// 128 37.0 and 27.4, 24 over 256 27.6 and 25.1; in two launches 23.0, 27.8 and 25.5).
constexpr int kShares = 8;                   // of the probability rows, one after the other (as in the kernel that adds them alone)
template <int MAX, bool ROWS>
__global__ __launch_bounds__(kThreads) void select_sums_kernel(ScoreSums a, float* __restrict__ score, const int64_t* __restrict__ ctx_off,
                                                               int64_t total_ctx, const int64_t* __restrict__ sel_off, int64_t total_sel,
                                                               int32_t* __restrict__ sel_idx, int32_t* __restrict__ sel_row,
                                                               int32_t* __restrict__ sel_pos) {
  __shared__ SelectLds lds;
  __shared__ __align__(16) float s[ROWS ? scoring::kSumRowTokens : scoring::kSumTokens];
  const int tid = threadIdx.x, total = (int)total_ctx;           // (at most the size of s)
  const int64_t p0 = min(max(a.probe_off[0], (int64_t)0), a.total_probe);
  const int64_t p1 = min(max(a.probe_off[1], p0), a.total_probe);
  const int64_t end = ctx_off[1];                                // tokens from here on have no score
  const float n = (float)((p1 - p0) * a.H);
  auto put = [&](int j, float sum) {
    const float v = p1 > p0 ? sum / n : 0.f;
    s[j] = v;
    if (j < end) score[j] = v;
  };
  if constexpr (ROWS) {
    float* part = reinterpret_cast<float*>(lds.list);            // [share][token]
    static_assert(kShares * scoring::kSumRowTokens <= kStage, "within the list");
    static_assert(kThreads / scoring::kSumRowTokens * 4 == kShares, "four shares to a thread at most");
    int width = 64;                                              // tokens side by side; the threads behind them take other shares
    while (width < total) width *= 2;
    const int j = tid % width, groups = kThreads / width;
    const int r0 = (int)(p0 * a.H), r1 = (int)(p1 * a.H), share = (r1 - r0 + kShares - 1) / kShares;
    const int group = __builtin_amdgcn_readfirstlane(tid / width), at = min(j, total - 1);       // (a wave is in one group)
    // S shares, and R rows of each, on their way together; row numbers are a wave's, so that a load costs no vector instruction more
    auto add = [&](auto s_c, auto r_c) {
      constexpr int S = decltype(s_c)::value, R = decltype(r_c)::value;
      float acc[S];
#pragma unroll
      for (int i = 0; i < S; ++i) acc[i] = 0.f;
      for (int r = 0; r < share; r += R) {
        float p[S][R];
#pragma unroll
        for (int i = 0; i < S; ++i)
#pragma unroll
          for (int u = 0; u < R; ++u) p[i][u] = (a.sums + max(min(r0 + (group + i * groups) * share + r + u, r1 - 1), 0) * total)[at];
#pragma unroll
        for (int i = 0; i < S; ++i) {
          const int first = r0 + (group + i * groups) * share + r, last = min(first - r + share, r1);
#pragma unroll
          for (int u = 0; u < R; ++u) acc[i] += first + u < last ? p[i][u] : 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < S; ++i)
        if (j < total) part[(group + i * groups) * total + j] = acc[i];
    };
    auto of_shares = [&](auto s_c) {
      if (share <= 4) add(s_c, std::integral_constant<int, 4>{});
      else if (share <= 8 || (share > 12 && share <= 16)) add(s_c, std::integral_constant<int, 8>{});
      else if (share <= 10) add(s_c, std::integral_constant<int, 10>{});
      else add(s_c, std::integral_constant<int, 12>{});
    };
    if (group < kShares) {
      if (groups >= kShares) of_shares(std::integral_constant<int, 1>{});
      else if (2 * groups == kShares) of_shares(std::integral_constant<int, 2>{});
      else of_shares(std::integral_constant<int, 4>{});
    }
    __syncthreads();
    if (tid < total) {
      float acc = 0.f;
#pragma unroll
      for (int w = 0; w < kShares; ++w) acc += part[w * total + tid];
      put(tid, acc);
    }
  } else {
    constexpr int U = MAX;                                       // tokens of a thread, kThreads apart
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.f;
#pragma unroll 8
    for (int g = 0; g < a.Hkv; ++g)
#pragma unroll
      for (int u = 0; u < U; ++u) acc[u] += a.sums[(int64_t)g * total + min(tid + u * kThreads, total - 1)];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (tid + u * kThreads < total) put(tid + u * kThreads, acc[u]);
  }
  __syncthreads();
  const int64_t c0 = min(max(ctx_off[0], (int64_t)0), total_ctx), c1 = min(max(end, c0), total_ctx);
  const int64_t o0 = min(max(sel_off[0], (int64_t)0), total_sel), o1 = min(max(sel_off[1], o0), total_sel);
  const int T = (int)(c1 - c0), N = (int)min((int64_t)T, o1 - o0);
  if (N <= 0) return;
  int seg = (T + kThreads - 1) / kThreads;
  if (seg > 1) seg = (seg + 3) & ~3;
  if (MAX == 1 || seg > 1) select_request<MAX>(lds, s + c0, c0, T, N, seg, o0, 0, sel_idx, sel_row, sel_pos);
  else select_request<1>(lds, s + c0, c0, T, N, seg, o0, 0, sel_idx, sel_row, sel_pos);
}

// Offline anchors: Top-N of a chunk, then its key and value rows, by the workgroup that selected them.  Bound by latency: the
// offsets of up to kAnchorChunks chunks travel as kernel arguments (3.6 of the 4 KB a launch can have), so that no copy to
// the device stands in front of the first kernel and no launch between the selection and the gather.  Whole extraction,
// us, with four operations on the stream and now: 64 chunks of 512, 26 rows each, 46 and 27; 4 chunks of 64 40 and 27.
constexpr int kAnchorChunks = 448, kFewChunks = 64;              // (few: half a kilobyte of arguments to hand over, not 3.6)
template <int N>
struct AnchorChunks {
  int32_t ctx[N + 1], sel[N + 1];                                // inside the totals (at most 2^30 rows)
};

template <int MAX, int CHUNKS>
__global__ __launch_bounds__(kThreads) void select_gather_kernel(const float* __restrict__ score, AnchorChunks<CHUNKS> ch,
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
  const int64_t out = o0 * vec_per_row;
  const int items = N * vec_per_row;                             // (at most kGatherVecs)
  for (int i0 = tid; i0 < items; i0 += 4 * kThreads) {
    u32x4 kk[4], vv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = min(i0 + u * kThreads, items - 1), m = i / vec_per_row;
      const int64_t src = (c0 + (N < T ? lds.list[m] : m)) * vec_per_row + (i - m * vec_per_row);
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
  // (with the choice by length inside one kernel: 731 tokens 4.2 us both ways, 5000 6.3 so and 6.5, 8192 6.8 and 6.7).
  if (total_ctx <= kThreads) QCF_LAUNCH(1);
  else if (total_ctx <= 4 * kThreads) QCF_LAUNCH(4);
  else if (total_ctx <= 8 * kThreads) QCF_LAUNCH(8);
  else if (total_ctx <= 32 * kThreads) QCF_LAUNCH(32);
  else QCF_LAUNCH(0);
#undef QCF_LAUNCH
  return check_launch("select");
}

qcf_status launch_select_sums(const ScoreSums& sums, float* score, const int64_t* ctx_off, int64_t total_ctx, const int64_t* sel_off,
                              int64_t total_sel, int32_t* sel_idx, int32_t* sel_row, int32_t* sel_pos, hipStream_t st) {
#define QCF_LAUNCH(MAX, ROWS) \
  select_sums_kernel<MAX, ROWS><<<dim3(1), dim3(kThreads), 0, st>>>(sums, score, ctx_off, total_ctx, sel_off, total_sel, sel_idx, sel_row, sel_pos)
  if (sums.rows) QCF_LAUNCH(1, true);
  else if (total_ctx <= kThreads) QCF_LAUNCH(1, false);
  else QCF_LAUNCH(4, false);
#undef QCF_LAUNCH
  return check_launch("select");
}

// A workgroup copies what its chunk selected up to this many 16-byte vectors of keys (64 rows of 8 heads of 128); with more
// the copy is a launch over all of them (64 chunks of 1024, 128 rows each: 56 us by the workgroups, 44 with the launch; 64
// rows each: 43 both ways).
constexpr int64_t kGatherVecs = 8192;
static_assert(kGatherVecs <= kStage, "the rows are read from the one window that they leave in");

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
  // one launch for the chunks from `first` on, as many as its arguments hold
  auto launch = [&](int32_t first, auto chunks_c) {
    constexpr int CHUNKS = decltype(chunks_c)::value;
    const int n = std::min(CHUNKS, n_chunks - first);
    AnchorChunks<CHUNKS> ch;
    for (int i = 0; i <= n; ++i) {
      ch.ctx[i] = (int32_t)ctx(first + i);
      ch.sel[i] = (int32_t)sel(first + i);
    }
#define QCF_LAUNCH(MAX)                                                                              \
  select_gather_kernel<MAX, CHUNKS><<<dim3((unsigned)n), dim3(kThreads), 0, st>>>(                   \
      score, ch, static_cast<const u32x4*>(k), static_cast<const u32x4*>(v), vec_per_row, rows,      \
      gather ? static_cast<u32x4*>(k_out) : nullptr, static_cast<u32x4*>(v_out))
    if (longest <= kThreads) QCF_LAUNCH(1);
    else if (longest <= 8 * kThreads) QCF_LAUNCH(8);
    else if (longest <= 32 * kThreads) QCF_LAUNCH(32);
    else QCF_LAUNCH(0);
#undef QCF_LAUNCH
    return check_launch("anchor select");
  };
  if (n_chunks <= kFewChunks) QCF_TRY(launch(0, std::integral_constant<int, kFewChunks>{}));
  else
    for (int32_t first = 0; first < n_chunks; first += kAnchorChunks) QCF_TRY(launch(first, std::integral_constant<int, kAnchorChunks>{}));
  return gather ? QCF_OK : launch_gather(L, k, v, rows, total_sel, total_ctx, k_out, v_out, st);
}

}  // namespace qcf
