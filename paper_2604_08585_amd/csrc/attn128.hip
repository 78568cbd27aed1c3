// Step 6 for bf16 heads of 128, long launches: 64 rows to a wave, four waves to a workgroup, one wave to a SIMD (the rule
// that chooses between this and the kernel of attn.hip, with both sides measured, is in attn_layout.h; layouts and arithmetic
// are the same, with the differences below).
//
// A key or value fragment read from LDS feeds two MFMAs instead of one, and a workgroup streams every tile for 256 rows.
// A wave alone on its SIMD issues everything itself: an MFMA takes 32 cycles of the matrix unit but blocks the wave for
// about 10, every other instruction for 4.6, an exponential for 8.5 (timed with loops of one MFMA and n others: up to four
// others are free, eight make 47 cycles).  So the loop is bound by the number of its instructions: 203 to 211 per half tile
// (32 tokens x 64 rows, 32 MFMAs), about 1650 cycles.  Hence
//   - no maximum: exponentials are taken against a reference point that only moves when a sum shows it too low (8 % of the
//     instructions; with the maximum, its exchange between the lane halves and the choice of the reference 2640 us, below);
//   - the argument, the exponential and the sum of an element are three MFMAs apart, and LDS is waited for four times per
//     half tile, for fragments requested eight MFMAs earlier;
//   - four tiles of keys and of values in LDS, loads on their way for a tile and a half, one barrier per tile;
//   - logits in vector registers, outputs (128) in accumulation registers, 248 + 128 in all: see pv().
// 4915 rows x 64 heads over 32768 tokens: 2468 us with 128 rows to a workgroup, 2262 here (1.16 PFLOP/s at 1.85 GHz; the
// matrix unit is busy 62 % of the cycles).  The same loop with the compiler's choice of registers (copies between the two
// kinds) took 2730.
#include <utility>

#include "attn_common.h"

namespace qcf {
namespace attn {
namespace {

constexpr int D = 128, KS = D / 16, DT = D / 32;
constexpr int kRow = 2 * D, kTile = kBKV * kRow;       // bytes of a staged token row, of a key or value tile
constexpr int kRing = 4;                               // tiles of each kept in LDS
constexpr int kRB = 2;                                 // 32-row blocks of a wave
constexpr int kWgRows = 4 * 32 * kRB;
static_assert(kWgRows == kWideRows, "four waves");
constexpr float kK2 = AttnTile<D>::K2;

constexpr float kUnseen = -3.0e38f;
constexpr float kCap = 256.f;                          // of 16 probabilities

#define QCF_INLINE __attribute__((always_inline))

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>): a loop body too large for the unroller's limit
template <int... I, class F>
__device__ __forceinline__ void each_of(std::integer_sequence<int, I...>, F&& f) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) { each_of(std::make_integer_sequence<int, N>{}, f); }
#define QCF_INT(x) std::integral_constant<int, (x)>{}
// f of the constants FROM .. TO - 1
template <int FROM, int TO, class F>
__device__ __forceinline__ void span(std::integral_constant<int, FROM>, std::integral_constant<int, TO>, F& f) {
  if constexpr (FROM < TO) {
    f(std::integral_constant<int, FROM>{});
    span(std::integral_constant<int, FROM + 1>{}, std::integral_constant<int, TO>{}, f);
  }
}

__global__ __launch_bounds__(256, 1) void attn128_kernel(AttnArgs a) {
  static_assert(kOrderLds <= 2 * kRing * kTile, "ordered_unit works in the tiles' LDS");
  extern __shared__ __align__(256) unsigned char smem[];      // (fragment addresses are formed with XORs below 256)
  int* s_vis_max = reinterpret_cast<int*>(smem + 2 * kRing * kTile);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5, l32 = lane & 31;
  const int BR = a.block_rows;
  const uint32_t lds_k = lds_offset_of(smem);

  const int g = (int)(blockIdx.x % a.Hkv);
  const int unit = (int)(blockIdx.x / a.Hkv);
  int seg = unit % a.n_seg_max, blk = a.n_row_blocks - 1 - unit / a.n_seg_max;
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
  const int64_t c0 = min(max(a.ctx_off[b], (int64_t)0), a.total_ctx);
  const int64_t c1 = min(max(a.ctx_off[b + 1], c0), a.total_ctx);
  const int T = (int)(c1 - c0);
  const int64_t p0 = a.ctx_pos0 ? a.ctx_pos0[b] : 0;

  // this lane's rows: wave * 64 + 32 rb + l32.  (Formed where they are needed: registers are short in between.)
  struct Row { int64_t sel; int head; bool ok; };
  auto row_of = [&](int l, int rb) QCF_INLINE {
    const int r = wave * 32 * kRB + 32 * rb + l;
    const int64_t sel = s0 + (int64_t)wg * BR + r / a.G;
    return Row{sel, g * a.G + r % a.G, sel < s1};
  };
  int vis[kRB], wave_vis_max = 0, wave_vis_min = 0x7fffffff;
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
    const Row row = row_of(l32, rb);
    vis[rb] = 0;
    if (row.ok) vis[rb] = (int)min((int64_t)T, max((int64_t)0, (int64_t)a.sel_pos[row.sel] - p0 + 1));
    wave_vis_max = max(wave_vis_max, vis[rb]);
    wave_vis_min = min(wave_vis_min, row.ok ? vis[rb] : 0x7fffffff);
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
    wave_vis_max = max(wave_vis_max, __shfl_xor(wave_vis_max, d, 64));
    wave_vis_min = min(wave_vis_min, __shfl_xor(wave_vis_min, d, 64));
  }
  wave_vis_max = __builtin_amdgcn_readfirstlane(wave_vis_max);
  wave_vis_min = __builtin_amdgcn_readfirstlane(wave_vis_min);
  if (lane == 0) s_vis_max[wave] = wave_vis_max;
  __syncthreads();
  const int wg_vis_max = max(max(s_vis_max[0], s_vis_max[1]), max(s_vis_max[2], s_vis_max[3]));
  const int n_tiles = (wg_vis_max + kBKV - 1) / kBKV;
  const bool split = n_tiles > a.seg_tiles;
  if (seg > 0 && seg * a.seg_tiles >= n_tiles) return;      // this block has fewer segments
  const int t_end = n_tiles - seg * a.seg_tiles;
  const int t_begin = max(0, t_end - a.seg_tiles);
  if (n_tiles == 0) {                 // nothing visible to any row of the block
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb) {
      const Row row = row_of(l32, rb);
      if (!row.ok) continue;
      bf16_t* op = static_cast<bf16_t*>(a.o) + (row.sel * a.H + row.head) * D + D / 2 * hf;
#pragma unroll
      for (int i = 0; i < D / 16; ++i) *reinterpret_cast<u32x4*>(op + 8 * i) = u32x4{0u, 0u, 0u, 0u};
      if (a.lse && hf == 0) a.lse[row.sel * a.H + row.head] = -INFINITY;
    }
    return;
  }

  // Tile loads: instruction i of wave w fills rows 16*i + 4*w .. +3 (1 KB) of a tile, the keys of tile `it` of this unit
  // in slot it % kRing of their ring, the values likewise.  Past the last tile that one is loaded again, so that every
  // iteration issues as many loads.  Tokens past the end of the context are clamped (their probabilities are zero).
  const uint32_t row_bytes = (uint32_t)a.Hkv * kRow;
  const char* kg = reinterpret_cast<const char*>(static_cast<const bf16_t*>(a.k) + (c0 * a.Hkv + g) * D);
  const char* vg = reinterpret_cast<const char*>(static_cast<const bf16_t*>(a.v) + (c0 * a.Hkv + g) * D);
  const int ld_row = 4 * wave + lane / 16;
  const uint32_t ld_kchunk = (uint32_t)(k_slot<D>(lane % 16, ld_row) * 16), ld_vchunk = (uint32_t)(v_slot<D>(lane % 16, ld_row) * 16);
  uint32_t koff[4], voff[4];
  auto set_offsets = [&](uint32_t (&off)[4], uint32_t chunk, int rows) QCF_INLINE {
#pragma unroll
    for (int i = 0; i < 4; ++i) off[i] = (uint32_t)min(16 * i + ld_row, rows - 1) * row_bytes + chunk;
  };
  set_offsets(koff, ld_kchunk, kBKV);
  set_offsets(voff, ld_vchunk, kBKV);
  const int whole = T / kBKV;                                    // the context's whole tiles
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((int)(lds_k + (uint32_t)wave * 1024));
  // the next tile to load of each kind; the clamped offsets of a partial tile stay (every later load is of that tile)
  const uint32_t tile_bytes = kBKV * row_bytes;
  const char* k_at = kg + (int64_t)t_begin * tile_bytes;
  const char* v_at = vg + (int64_t)t_begin * tile_bytes;
  int k_next_t = t_begin, v_next_t = t_begin;
  auto k_tile = [&]() QCF_INLINE {
    if (k_next_t == whole) set_offsets(koff, ld_kchunk, T - whole * kBKV);
    const char* at = k_at;
    const bool more = k_next_t + 1 < t_end;
    k_at += more ? tile_bytes : 0u;
    k_next_t += more ? 1 : 0;
    return at;
  };
  auto v_tile = [&]() QCF_INLINE {
    if (v_next_t == whole) set_offsets(voff, ld_vchunk, T - whole * kBKV);
    const char* at = v_at;
    const bool more = v_next_t + 1 < t_end;
    v_at += more ? tile_bytes : 0u;
    v_next_t += more ? 1 : 0;
    return at;
  };
  auto slot = [&](int it) QCF_INLINE { return (uint32_t)((it & (kRing - 1)) * kTile); };
  auto load_k1 = [&](uint32_t at, auto i_c, const char* tile) QCF_INLINE {
    load_to_lds_const<decltype(i_c)::value * 4096>(tile, koff[decltype(i_c)::value], lds_wave + at);
  };
  auto load_v1 = [&](uint32_t at, auto i_c, const char* tile) QCF_INLINE {
    load_to_lds_const<kRing * kTile + decltype(i_c)::value * 4096>(tile, voff[decltype(i_c)::value], lds_wave + at);
  };
  std::integral_constant<int, 0> n0;
  std::integral_constant<int, 1> n1;
  std::integral_constant<int, 2> n2;
  std::integral_constant<int, 3> n3;
  auto load_k = [&](int it) QCF_INLINE {
    const char* t = k_tile();
    load_k1(slot(it), n0, t); load_k1(slot(it), n1, t); load_k1(slot(it), n2, t); load_k1(slot(it), n3, t);
  };
  auto load_v = [&](int it) QCF_INLINE {
    const char* t = v_tile();
    load_v1(slot(it), n0, t); load_v1(slot(it), n1, t); load_v1(slot(it), n2, t); load_v1(slot(it), n3, t);
  };
  load_k(0);
  load_v(0);
  load_k(1);
  load_k(2);
  load_v(1);

  bf16x8 qf[kRB][KS];                // row 32 rb + l32, elements 16*ks + 8*hf .. +7
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
    const Row row = row_of(l32, rb);
    const bf16_t* qp = static_cast<const bf16_t*>(a.q) + ((row.ok ? row.sel : s0) * a.H + row.head) * D + 8 * hf;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u32x4 t = *reinterpret_cast<const u32x4*>(qp + 16 * ks);
      if (!row.ok) t = u32x4{0u, 0u, 0u, 0u};
      qf[rb][ks] = __builtin_bit_cast(bf16x8, t);
    }
  }

  // LDS addresses of this lane's first fragments in slot 0; key fragment ks is at ^ 32 ks, that of output slice dt at ^ 64 dt
  const uint32_t kofs = lds_k + l32 * kRow + k_slot<D>(hf, l32) * 16;
  uint32_t vofs;
  {
    const int vq = 4 * ((lane >> 4) & 1) + (lane & 3);
    const int d0 = 16 * (vq & 1) + 4 * (vq >> 1);
    const int vrow = 4 * hf + ((lane & 15) >> 2);
    vofs = lds_k + kRing * kTile + vrow * kRow + v_slot<D>(d0 / 8, vrow) * 16 + (d0 & 4) * 2;
  }

  floatx16 oacc[kRB][DT];            // in accumulation registers, see pv()
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) oacc[rb][dt] = floatx16{0};
  // Exponentials are taken against m_use (log2 units), which only moves when a lane's sum over a half tile passes kCap
  // (or is not a number): the division by the denominator makes the result independent of it, and no maximum is needed.
  // A row that has seen nothing yet has a reference point so low that its first visible token passes any cap.
  float m_use[kRB], l_run[kRB];
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) { m_use[rb] = kUnseen; l_run[rb] = 0.f; }

  floatx16 s_a[kRB], s_b[kRB];       // logits of the even and the odd half tiles
  u32x4 p_a[kRB][2], p_b[kRB][2];    // their probabilities: step s of 16 tokens
  u32x4 kf[4];                       // key fragments, up to four ahead
  shortx4 vlo[4], vhi[4];            // value fragments, up to four ahead

  constexpr uint32_t kHalf = 32 * kRow;
  auto read_k = [&](uint32_t at, int ks) QCF_INLINE { kf[ks & 3] = lds_read16((kofs + at) ^ (uint32_t)(32 * ks)); };     // at: slot and half
  auto read_v = [&](uint32_t at, int idx) QCF_INLINE {
    const uint32_t addr = ((vofs + at) ^ (uint32_t)(64 * (idx & 3))) + (uint32_t)(16 * (idx >> 2) * kRow);
    vlo[idx & 3] = lds_read_tr(addr);
    vhi[idx & 3] = lds_read_tr(addr + 8 * kRow);
  };
  // output slice dt += values x probabilities.  The accumulators of the two products together exceed the vector registers,
  // and the compiler keeps both kinds in the same ones, so this one names accumulation registers itself.  The wait states
  // that the compiler would have put in are kept by the order instead: an operand written by a vector instruction needs two
  // instructions before the MFMA (the fragment is formed, if it is moved at all, before the two logit MFMAs in front of its
  // first use; the probabilities half a tile earlier), and other uses of oacc are fenced (`settle`: an MFMA's result may be
  // read 11 wait states later).  tests/test_attn128_waits.py looks for both in the assembly.
  bf16x8 vf[2];
  auto v_form = [&](int idx) QCF_INLINE {
    u32x4 t = __builtin_bit_cast(u32x4, __builtin_shufflevector(vlo[idx & 3], vhi[idx & 3], 0, 1, 2, 3, 4, 5, 6, 7));
    asm volatile("" : "+v"(t));
    vf[idx & 1] = __builtin_bit_cast(bf16x8, t);
  };
  auto pv = [&](int rb, int idx, const u32x4 (&p)[kRB][2]) QCF_INLINE {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(oacc[rb][idx & 3]) : "v"(vf[idx & 1]), "v"(p[rb][idx >> 2]));
  };
  auto settle = [&]() QCF_INLINE {
    asm volatile("s_nop 15\n\ts_nop 7" : "+a"(oacc[0][0]), "+a"(oacc[0][1]), "+a"(oacc[0][2]), "+a"(oacc[0][3]),
                 "+a"(oacc[1][0]), "+a"(oacc[1][1]), "+a"(oacc[1][2]), "+a"(oacc[1][3]));
  };

  // One half tile (32 tokens from kv0 on): softmax of `cur` into `pc`, while the matrix unit computes the logits of the
  // next half (keys at k_now) and the output's share of the previous one (values at v_now, probabilities `pp`); the first
  // fragments of the halves after those (k_next, v_next) are requested at the end.
  auto half = [&](auto pv_c, uint32_t k_now, uint32_t k_next, uint32_t v_now, uint32_t v_next, floatx16 (&cur)[kRB],
                  floatx16 (&nxt)[kRB], u32x4 (&pc)[kRB][2], const u32x4 (&pp)[kRB][2], int kv0, auto load) QCF_INLINE {
    constexpr bool PV = decltype(pv_c)::value;
    if (kv0 + 32 > wave_vis_min) {
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb) {
        const int left = vis[rb] - kv0 - 4 * hf;
#pragma unroll
        for (int v = 0; v < 16; ++v) cur[rb][v] = (8 * (v >> 2) + (v & 3) < left) ? cur[rb][v] : -INFINITY;
      }
    }
    float sum[kRB];
    // element e of the lane's 32 in three steps, so that nothing waits for the step before: argument, exponential, sum.
    // Element e is register 2 (e / 4) + e % 2 of row block e / 2 % 2.
    float arg[32], ex[32];
    auto step_arg = [&](auto e_c) QCF_INLINE {
      constexpr int e = decltype(e_c)::value, rb = (e >> 1) & 1, v = 2 * (e >> 2) + (e & 1);
      arg[e] = __builtin_fmaf(cur[rb][v], kK2, -m_use[rb]);
      asm volatile("" : "+v"(arg[e]));                 // (the steps stay where they are written)
    };
    auto step_exp = [&](auto e_c) QCF_INLINE {
      constexpr int e = decltype(e_c)::value;
      ex[e] = __builtin_amdgcn_exp2f(arg[e]);
    };
    auto step_sum = [&](auto e_c) QCF_INLINE {
      constexpr int e = decltype(e_c)::value, rb = (e >> 1) & 1, v = 2 * (e >> 2) + (e & 1);
      sum[rb] = e == 2 * rb ? ex[e] : sum[rb] + ex[e];
      if constexpr (e & 1) {
        uint32_t pk = cvt_pk_bf16(ex[e - 1], ex[e]);
        asm volatile("" : "+v"(pk), "+v"(sum[rb]));
        pc[rb][v >> 3][(v & 7) >> 1] = pk;
      }
    };
    step_arg(n0);
    step_arg(n1);
    unrolled<32>([&](auto n_c) QCF_INLINE {
      constexpr int n = decltype(n_c)::value, j = n >> 2, w = n & 3;
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (n % 8 == 0) {                // fragments of the next eight MFMAs, all requested a good while ago
        __builtin_amdgcn_s_waitcnt(0xc07f);        // lgkmcnt(0)
        __builtin_amdgcn_sched_barrier(0);
        if (PV) { v_form(j); v_form(j + 1); }
      }
      if constexpr (w < 2) {
        if (j == 0) nxt[w] = floatx16{0};
        nxt[w] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[j & 3]), qf[w][j], nxt[w], 0, 0, 0);
      } else if constexpr (PV) {
        pv(w - 2, j, pp);
      }
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (n % 8 == 0) {                // request those of the eight after
#pragma unroll
        for (int u = 2; u < 4; ++u)
          if (j + u < KS) read_k(k_now, j + u);
          else read_k(k_next, j + u - KS);
      }
      if constexpr (n % 8 == 1) {
#pragma unroll
        for (int u = 2; u < 4; ++u) {
          const int idx = (n >> 3) * 2 + u;
          if (idx < 8) { if (PV) read_v(v_now, idx); }
          else read_v(v_next, idx - 8);
        }
      }
      step_exp(n_c);
      if constexpr (n < 30) step_arg(QCF_INT(n + 2));
      if constexpr (n > 0) step_sum(QCF_INT(n - 1));
      asm volatile("" : "+v"(ex[n]));                  // (not right behind the exponential, which would need a wait state)
      if constexpr (n == 6) load(n0);
      if constexpr (n == 13) load(n1);
      if constexpr (n == 20) load(n2);
      if constexpr (n == 27) load(n3);
    });
    step_sum(QCF_INT(31));
    __builtin_amdgcn_sched_barrier(0);
    if (__any(!(sum[0] <= kCap) || !(sum[1] <= kCap))) {       // a new reference point: this half's exponentials again
      settle();
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb) {
        // (with the tokens of the next half: the further the reference lags behind a row's maximum, the larger the rounding
        // errors of the probabilities that weigh most, those just above a power of two)
        const int left = vis[rb] - kv0 - 32 - 4 * hf;
        float mx = cur[rb][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, cur[rb][v]);
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, 8 * (v >> 2) + (v & 3) < left ? nxt[rb][v] : -INFINITY);
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        bool up = !(sum[rb] <= kCap);
        up |= (bool)__shfl_xor((int)up, 32, 64);
        const float m_new = up && mx > -INFINITY ? mx * kK2 : m_use[rb];
        const float alpha = m_new == m_use[rb] ? 1.f : m_use[rb] == kUnseen ? 0.f : __builtin_amdgcn_exp2f(m_use[rb] - m_new);
        m_use[rb] = m_new;
        sum[rb] = 0.f;
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          const float e0 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[rb][v], kK2, -m_new));
          const float e1 = __builtin_amdgcn_exp2f(__builtin_fmaf(cur[rb][v + 1], kK2, -m_new));
          sum[rb] += e0;
          sum[rb] += e1;
          pc[rb][v >> 3][(v & 7) >> 1] = cvt_pk_bf16(e0, e1);
        }
        l_run[rb] *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {              // (one after the other: few registers)
          __builtin_amdgcn_sched_barrier(0);
          asm volatile("" : "+a"(oacc[rb][dt]));
#pragma unroll
          for (int v = 0; v < 16; ++v) oacc[rb][dt][v] *= alpha;
          asm volatile("" : "+a"(oacc[rb][dt]));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      settle();
    }
    l_run[0] += sum[0];
    l_run[1] += sum[1];
  };
  std::true_type yes;
  std::false_type no;

  const int n_it = t_end - t_begin;
  const int wave_it = min(n_it, (wave_vis_max + kBKV - 1) / kBKV - t_begin);      // iterations with something to see
  // keys of tile it + 1 and values of tile it have landed; all waves are done with keys it - 1 and values it - 2
  auto next_tile = [&]() QCF_INLINE { asm volatile("s_waitcnt vmcnt(8)\n\ts_barrier" ::: "memory"); };
  int it = 0;
  if (wave_it > 0) {
    next_tile();
    read_k(0u, 0);
    read_k(0u, 1);
#pragma unroll
    for (int rb = 0; rb < kRB; ++rb) s_a[rb] = floatx16{0};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb)
        s_a[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[ks & 3]), qf[rb][ks], s_a[rb], 0, 0, 0);
      read_k(ks + 2 < KS ? 0u : kHalf, (ks + 2) & 7);
    }
    settle();
    // iteration `it`: tile t_begin + it
    const char *kt, *vt;
    auto lk = [&](auto i) QCF_INLINE { load_k1(slot(it + 3), i, kt); };
    auto lv = [&](auto i) QCF_INLINE { load_v1(slot(it + 2), i, vt); };
    kt = k_tile();
    half(no, kHalf, slot(1), 0u, 0u, s_a, s_b, p_a, p_b, t_begin * kBKV, lk);
    vt = v_tile();
    half(yes, slot(1), slot(1) + kHalf, 0u, kHalf, s_b, s_a, p_b, p_a, t_begin * kBKV + 32, lv);
#pragma unroll 1
    for (it = 1; it < wave_it; ++it) {
      next_tile();
      const uint32_t k0 = slot(it), k1 = slot(it + 1), v0 = slot(it), vm = slot(it - 1);
      const int kv0 = (t_begin + it) * kBKV;
      kt = k_tile();
      half(yes, k0 + kHalf, k1, vm + kHalf, v0, s_a, s_b, p_a, p_b, kv0, lk);
      vt = v_tile();
      half(yes, k1, k1 + kHalf, v0, v0 + kHalf, s_b, s_a, p_b, p_a, kv0 + 32, lv);
    }
    // the output's share of the last half (its first two fragments are there)
    const uint32_t vl = slot(it - 1) + kHalf;
#pragma unroll
    for (int idx = 2; idx < 4; ++idx) read_v(vl, idx);
#pragma unroll
    for (int idx = 0; idx < 8; ++idx) {
      v_form(idx);
      if (idx < 4) read_v(vl, idx + 4);
      asm volatile("s_nop 1");
#pragma unroll
      for (int rb = 0; rb < kRB; ++rb) pv(rb, idx, p_b);
    }
    settle();
  }
  for (; it < n_it; ++it) {              // the other waves' tiles
    next_tile();
    load_k(it + 3);
    load_v(it + 2);
  }
  __builtin_amdgcn_s_waitcnt(0);                        // (no load is on its way when the workgroup ends)

  // epilogue: output register v of slice dt is element 32*dt + 16*hf + v of this lane's row
  int l_end = l32;
  asm volatile("" : "+v"(l_end));
#pragma unroll
  for (int rb = 0; rb < kRB; ++rb) {
    const Row row = row_of(l_end, rb);
    const float l_tot = l_run[rb] + __shfl_xor(l_run[rb], 32, 64);
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    if (split) {
      // (fp32: bf16 would be rounded once more than in a whole block; 1229 rows over 8192 tokens 2.22e-3 off in the 2-norm
      // of the difference, 2.33e-3 with bf16)
      const int64_t row0 = (((int64_t)blk * a.Hkv + g) * a.n_seg_max + seg) * kWgRows + wave * 32 * kRB + 32 * rb;
      float* dst = static_cast<float*>(a.part_o) + row0 * D + (32 * hf + l_end) * 4;      // in register order
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
          const floatx16& o = oacc[rb][dt];
          *reinterpret_cast<float4*>(dst + (4 * dt + v / 4) * 256) = make_float4(o[v] * inv, o[v + 1] * inv, o[v + 2] * inv, o[v + 3] * inv);
        }
      if (hf == 0) a.part_lse[row0 + l_end] = l_tot > 0.f ? m_use[rb] + log2f(l_tot) : -INFINITY;
    } else if (row.ok) {
      bf16_t* dst = static_cast<bf16_t*>(a.o) + (row.sel * a.H + row.head) * D + 16 * hf;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int h8 = 0; h8 < 16; h8 += 8) {
          const floatx16& o = oacc[rb][dt];
          *reinterpret_cast<u32x4*>(dst + 32 * dt + h8) = mk4(cvt_pk_bf16(o[h8] * inv, o[h8 + 1] * inv), cvt_pk_bf16(o[h8 + 2] * inv, o[h8 + 3] * inv),
                                                             cvt_pk_bf16(o[h8 + 4] * inv, o[h8 + 5] * inv), cvt_pk_bf16(o[h8 + 6] * inv, o[h8 + 7] * inv));
        }
      if (a.lse && hf == 0) a.lse[row.sel * a.H + row.head] = natural_lse<true>(l_tot > 0.f ? m_use[rb] : -INFINITY, log2f(l_tot));
    }
  }
}

}  // namespace

size_t attn128_lds() { return (size_t)2 * kRing * kTile + 4 * sizeof(int); }

qcf_status run_attn128(const AttnArgs& a, int64_t n_wg, hipStream_t st) {
  static std::atomic<uint64_t> lds_ok{0};
  QCF_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(&attn128_kernel), attn128_lds(), lds_ok));
  attn128_kernel<<<dim3((unsigned)n_wg), dim3(256), attn128_lds(), st>>>(a);
  return check_launch("attn");
}

}  // namespace attn
}  // namespace qcf
