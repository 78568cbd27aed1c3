// Step 4: recompute Q/K/V of the selected tokens (Section 3.1 Phase 4 of the paper):
// [Q|K|V] = X_sel W_qkv^T, rotary embedding on Q and K at the tokens' absolute positions.
//
// The bf16 path is a 32x32x16-MFMA GEMM (both operands are contiguous along the contraction
// dimension) with a ring of LDS stages; a wave's outputs are whole heads, so the rotary partner of
// every element is in the same lane and the embedding is applied in the epilogue, which forms the
// rotation itself: the angle pos * theta_i is taken in turns, with the frequency split in two floats
// and the product's rounding error recovered by a fused multiply-add (a plain float32 product would be
// off by 1e-3 rad at 8K positions), reduced to its fraction and handed to the hardware sine and cosine
// (inputs in turns, errors far below a bf16 ulp).  Positions from 2^24 on are taken in two parts.
// The generic path (f32, or shapes the MFMA tiling does not cover) takes float64 angles: in the product's epilogue where it is
// small, otherwise in a second kernel that finds the raw product in the workspace; both also write the cache rows.
// qcf_recompute_qkv_scatter: the epilogue of the MFMA path also stores the K and V rows to their rows of the
// fused cache (step 5 of the path, otherwise a kernel of its own).
#include <type_traits>
#include <utility>

#include "gemm_args.h"
#include "gemm_plan.h"
#include "qcf_internal.h"

namespace qcf {
using namespace gemm;
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------------ generic path

// 64 x 64 outputs per workgroup, 4 x 4 per thread; the sums run over k in order.
template <typename T>
__global__ __launch_bounds__(256) void qkv_gemm_generic(const T* __restrict__ x, int64_t x_rows,
                                                        const int32_t* __restrict__ gather, int64_t M,
                                                        const T* __restrict__ w, int Kdim, int Ntot,
                                                        float* __restrict__ y) {
  __shared__ float sA[16][65];
  __shared__ float sB[16][65];
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const int64_t m0 = (int64_t)blockIdx.x * 64;
  const int n0 = blockIdx.y * 64;
  float acc[4][4] = {};
  const int lr = tid >> 2;            // 0..63: tile row loaded by this thread
  const int lc = (tid & 3) * 4;       // 0,4,8,12: first k of its 4 elements
  int64_t arow = -1;
  if (m0 + lr < M) {
    const int64_t idx = gather ? (int64_t)gather[m0 + lr] : m0 + lr;
    if (idx >= 0 && idx < x_rows) arow = idx;
  }
  const int brow = (n0 + lr < Ntot) ? n0 + lr : -1;
  for (int k0 = 0; k0 < Kdim; k0 += 16) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int kk = k0 + lc + c;
      sA[lc + c][lr] = (arow >= 0 && kk < Kdim) ? Elem<T>::load(x + arow * Kdim + kk) : 0.f;
      sB[lc + c][lr] = (brow >= 0 && kk < Kdim) ? Elem<T>::load(w + (int64_t)brow * Kdim + kk) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float av[4], bv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) { av[i] = sA[kk][ty * 4 + i]; bv[i] = sB[kk][tx * 4 + i]; }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] += av[i] * bv[j];
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n < Ntot) y[m * Ntot + n] = acc[i][j];
    }
  }
}

// Where the heads of a projection row go on the generic path, and its rotation.
template <typename T>
struct RopeOut {
  const int32_t* pos;
  double neg2_over_d_log2base;
  int H, Hkv, D, style;
  T* q;
  T* k;
  T* v;
  const int32_t* dst_rows;       // K and V rows also go to the fused cache
  T* k_fused;
  T* v_fused;
  int64_t fused_rows;
  // columns of pair i of a head
  __device__ __forceinline__ int first(int i) const { return style == 0 ? i : 2 * i; }
  __device__ __forceinline__ int second(int i) const { return style == 0 ? i + D / 2 : 2 * i + 1; }
  __device__ __forceinline__ bool rotated(int head) const { return head < H + Hkv; }
  __device__ __forceinline__ float2 factor(int64_t m, int i) const {
    return rotary_pair((double)pos[m], neg2_over_d_log2base, i);
  }
  // head `head` of output row m (null: not wanted) and of its row of the cache (null: none)
  __device__ __forceinline__ T* out(int64_t m, int head) const {
    if (head < H) return q ? q + (m * H + head) * D : nullptr;
    T* base = head < H + Hkv ? k : v;
    return base ? base + (m * Hkv + (head - H) % Hkv) * D : nullptr;
  }
  __device__ __forceinline__ T* cache(int64_t m, int head) const {
    if (head < H || !dst_rows) return nullptr;
    const int64_t row = dst_rows[m];
    if (row < 0 || row >= fused_rows) return nullptr;
    return (head < H + Hkv ? k_fused : v_fused) + (row * Hkv + (head - H) % Hkv) * D;
  }
};

// The same product (same sums in the same order) with 16 x 16 outputs per workgroup, one per thread, for launches
// whose 64 x 64 tiles would leave most compute units idle.  Bound by latency there: the next 64 elements of the
// contraction are on their way while 64 are used.  M 77, K 256, N 512 in f32: 38 us with 64 x 64 tiles, 11 us here.
// ROPE: the 16 columns are 8 rotary pairs of a head, the columns of a pair 8 threads apart, and the results leave rotated and
// in the element type; the angles are taken in float64 while the first loads are on their way.  The same product 6.3 us, 4.9 + 3.3
// with a kernel of its own for the rotation.
template <typename T, bool ROPE>
__global__ __launch_bounds__(256) void qkv_gemm_small_generic(const T* __restrict__ x, int64_t x_rows,
                                                              const int32_t* __restrict__ gather, int64_t M,
                                                              const T* __restrict__ w, int Kdim, int Ntot,
                                                              float* __restrict__ y, RopeOut<T> ro) {
  constexpr int KC = 64, LD = KC + 4;            // (rows 4 banks apart: 16-byte reads of 16 rows touch every bank once)
  __shared__ __align__(16) float sA[16 * LD];
  __shared__ __align__(16) float sB[16 * LD];
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const int64_t m0 = (int64_t)blockIdx.x * 16;
  const int n0 = blockIdx.y * 16;
  const int head = ROPE ? n0 / ro.D : 0, pair0 = ROPE ? n0 % ro.D / 2 : 0;       // (D is a multiple of 16)
  auto column = [&](int c) {                     // weight row of tile column c
    if (!ROPE) return n0 + c;
    return head * ro.D + (c < 8 ? ro.first(pair0 + c) : ro.second(pair0 + c - 8));
  };
  const int lr = tid >> 4, lc = (tid & 15) * 4;  // row and first k of the four elements this thread brings
  int64_t arow = -1;
  if (m0 + lr < M) {
    const int64_t idx = gather ? (int64_t)gather[m0 + lr] : m0 + lr;
    if (idx >= 0 && idx < x_rows) arow = idx;
  }
  const int brow = column(lr) < Ntot ? column(lr) : -1;
  float a4[4], b4[4];
  auto fetch = [&](int k0) {                     // (Kdim is a multiple of 4 here)
#pragma unroll
    for (int c = 0; c < 4; ++c) a4[c] = b4[c] = 0.f;
    if (k0 + lc < Kdim) {
      if (arow >= 0) Quad<T>::load(x + arow * Kdim + k0 + lc, a4);
      if (brow >= 0) Quad<T>::load(w + (int64_t)brow * Kdim + k0 + lc, b4);
    }
  };
  fetch(0);
  float2 cs = make_float2(1.f, 0.f);
  if (ROPE && ro.rotated(head) && m0 + ty < M) cs = ro.factor(m0 + ty, pair0 + (tx & 7));
  float acc = 0.f;
  for (int k0 = 0; k0 < Kdim; k0 += KC) {
    __syncthreads();
    *reinterpret_cast<float4*>(sA + lr * LD + lc) = make_float4(a4[0], a4[1], a4[2], a4[3]);
    *reinterpret_cast<float4*>(sB + lr * LD + lc) = make_float4(b4[0], b4[1], b4[2], b4[3]);
    __syncthreads();
    if (k0 + KC < Kdim) fetch(k0 + KC);
#pragma unroll
    for (int kk = 0; kk < KC; kk += 4) {
      const float4 av = *reinterpret_cast<const float4*>(sA + ty * LD + kk);
      const float4 bv = *reinterpret_cast<const float4*>(sB + tx * LD + kk);
      acc += av.x * bv.x;
      acc += av.y * bv.y;
      acc += av.z * bv.z;
      acc += av.w * bv.w;
    }
  }
  if constexpr (!ROPE) {
    if (m0 + ty < M && n0 + tx < Ntot) y[(m0 + ty) * Ntot + n0 + tx] = acc;
  } else {
    const float other = __shfl_xor(acc, 8, 64);
    float ra = acc, rb = acc;
    if (ro.rotated(head)) {
      const float a = tx < 8 ? acc : other, b = tx < 8 ? other : acc;
      turn_pair(a, b, cs, ra, rb);
    }
    const float r = tx < 8 ? ra : rb;
    if (m0 + ty >= M) return;
    T* dst = ro.out(m0 + ty, head);
    if (!dst) return;
    const int c = column(tx) - head * ro.D;
    Elem<T>::store(dst + c, r);
    if (T* fus = ro.cache(m0 + ty, head)) Elem<T>::store(fus + c, r);
  }
}

// One thread per (row, head slot, rotary pair); V heads are copied.  The angle is taken in float64 (cheaper here than
// a table from a launch of its own: 77 rows, 4 us less).
template <typename T>
__global__ __launch_bounds__(256) void qkv_rope_split_generic(const float* __restrict__ y, int64_t M, RopeOut<T> ro) {
  const int half = ro.D / 2;
  const int heads = ro.H + 2 * ro.Hkv;
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (gid >= M * heads * half) return;
  const int i = (int)(gid % half);
  const int hs = (int)((gid / half) % heads);
  const int64_t m = gid / ((int64_t)half * heads);
  const int ia = ro.first(i), ib = ro.second(i);
  const float* src = y + m * (int64_t)heads * ro.D + (int64_t)hs * ro.D;
  const float a = src[ia], b = src[ib];
  T* dst = ro.out(m, hs);
  if (!dst) return;
  float ra = a, rb = b;
  if (ro.rotated(hs)) turn_pair(a, b, ro.factor(m, i), ra, rb);
  Elem<T>::store(dst + ia, ra);
  Elem<T>::store(dst + ib, rb);
  if (T* fus = ro.cache(m, hs)) {
    Elem<T>::store(fus + ia, ra);
    Elem<T>::store(fus + ib, rb);
  }
}

// out = y (+ residual), stored in the element type (generic path of the plain linear map)
template <typename T>
__global__ __launch_bounds__(256) void linear_finish_generic(const float* __restrict__ y, const T* residual,
                                                             int64_t n, T* out) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float v = y[i];
  if (residual) v += Elem<T>::load(residual + i);
  Elem<T>::store(out + i, v);
}

// ------------------------------------------------------------------ RMSNorm and gated SiLU (HBM bound)

// One workgroup per row: every thread keeps its 16-byte vectors of the row in registers (up to kNormVecs),
// the sum of squares goes through the waves and LDS in a fixed order, then the row is scaled and stored.
constexpr int kNormVecs = 4;
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const T* x, const T* __restrict__ weight, float eps, int cols,
                                                      T* out) {
  constexpr int VEC = Elem<T>::kVec;
  __shared__ float red[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = blockIdx.x;
  const T* xr = x + row * cols;
  const int n_vec = cols / VEC;
  u32x4 raw[kNormVecs];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < kNormVecs; ++i) {
    const int v = tid + i * 256;
    if (v < n_vec) {
      raw[i] = *reinterpret_cast<const u32x4*>(xr + v * VEC);
      float f[VEC];
      Vec16<T>::unpack(raw[i], f);
#pragma unroll
      for (int e = 0; e < VEC; ++e) ss += f[e] * f[e];
    }
  }
  for (int v = tid + kNormVecs * 256; v < n_vec; v += 256) {       // longer rows: the tail is read twice
    float f[VEC];
    Vec16<T>::unpack(*reinterpret_cast<const u32x4*>(xr + v * VEC), f);
#pragma unroll
    for (int e = 0; e < VEC; ++e) ss += f[e] * f[e];
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) ss += __shfl_xor(ss, d, 64);
  if (lane == 0) red[wave] = ss;
  __syncthreads();
  const float scale = rsqrtf(((red[0] + red[1]) + (red[2] + red[3])) / (float)cols + eps);
  T* orow = out + row * cols;
  auto emit = [&](int v, const u32x4& r) {
    float f[VEC], g[VEC];
    Vec16<T>::unpack(r, f);
    Vec16<T>::unpack(*reinterpret_cast<const u32x4*>(weight + v * VEC), g);
#pragma unroll
    for (int e = 0; e < VEC; ++e) f[e] = f[e] * scale * g[e];
    *reinterpret_cast<u32x4*>(orow + v * VEC) = Vec16<T>::pack(f);
  };
#pragma unroll
  for (int i = 0; i < kNormVecs; ++i) {
    const int v = tid + i * 256;
    if (v < n_vec) emit(v, raw[i]);
  }
  for (int v = tid + kNormVecs * 256; v < n_vec; v += 256) emit(v, *reinterpret_cast<const u32x4*>(xr + v * VEC));
}

// silu(g) * u.  A true division: one reciprocal with a Newton step in its place made the gate / up product 1 % faster
// (1229 rows, K 4096, F 14336: 241.7 us, 244.4 with the division) but flushed quotients whose divisor passes 2^126, i.e.
// g below -87.3, where they are still normal numbers.
__device__ __forceinline__ float silu_mul(float g, float u) { return g / (1.f + __expf(-g)) * u; }

// out[m, f] = silu(gate_up[m, f]) * gate_up[m, F + f]; one 16-byte output vector per thread
template <typename T>
__global__ __launch_bounds__(256) void swiglu_kernel(const T* __restrict__ gate_up, int64_t M, int F,
                                                     T* __restrict__ out) {
  constexpr int VEC = Elem<T>::kVec;
  const int per_row = F / VEC;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= M * per_row) return;
  const int64_t m = i / per_row;
  const int c = (int)(i - m * per_row) * VEC;
  float g[VEC], u[VEC];
  Vec16<T>::unpack(*reinterpret_cast<const u32x4*>(gate_up + m * 2 * F + c), g);
  Vec16<T>::unpack(*reinterpret_cast<const u32x4*>(gate_up + m * 2 * F + F + c), u);
#pragma unroll
  for (int e = 0; e < VEC; ++e) g[e] = silu_mul(g[e], u[e]);
  *reinterpret_cast<u32x4*>(out + m * F + c) = Vec16<T>::pack(g);
}

// ------------------------------------------------------------------ MFMA path (bf16)

constexpr int kRho16 = 64;               // rotary pairs of a head, at most
constexpr size_t kRhoBytes = 2 * kRho16 * sizeof(float2);      // their frequencies (fill_rho)

// Where a 128-column block of the product goes.
struct OutTile {
  bf16_t* out;
  bf16_t* fused;          // second destination, addressed through dst_rows (K and V tiles of the fused call)
  int out_cols, out_col0;
  bool rotate;
};
template <int EPI>
__device__ __forceinline__ OutTile out_tile_of(const QkvArgs& a, int block) {
  OutTile o;
  o.rotate = is_rope(EPI);
  o.fused = nullptr;
  if (EPI == kGlu) {
    o.out = a.q; o.out_cols = a.glu; o.out_col0 = block * (kBN / 2);
    return o;
  }
  const int col0 = block * kBN;
  const int q_cols = a.H * a.D, kv_cols = a.Hkv * a.D;
  if (col0 < q_cols) { o.out = a.q; o.out_cols = q_cols; o.out_col0 = col0; }
  else if (col0 < q_cols + kv_cols) { o.out = a.k; o.fused = a.k_fused; o.out_cols = kv_cols; o.out_col0 = col0 - q_cols; }
  else { o.out = a.v; o.fused = a.v_fused; o.out_cols = kv_cols; o.out_col0 = col0 - q_cols - kv_cols; o.rotate = false; }
  return o;
}
// first weight row of a 128-column block, and the distance from it to the weight row of column c
template <int EPI>
__device__ __forceinline__ int64_t block_w_row(int block) {
  return (int64_t)block * (EPI == kGlu ? kBN / 2 : kBN);
}
template <int EPI>
__device__ __forceinline__ uint32_t block_w_step(const QkvArgs& a, int c) {
  return (uint32_t)((EPI == kGlu && c >= kBN / 2) ? a.glu + c - kBN / 2 : c);
}

// Rotary frequencies in turns per position, theta_i / (2 pi) = 2^(i * c) / (2 pi), for the d/2 pairs of a head:
// computed in float64 and kept as two floats, high + low; kRho16 entries further the fraction of 2^16 times each
// (written by 64 threads before the barrier that precedes the epilogue).
__device__ __forceinline__ float2 two_floats(double x) {
  const float hi = (float)x;
  return make_float2(hi, (float)(x - (double)hi));
}
__device__ __forceinline__ void fill_rho(const QkvArgs& a, float2* sRho, int i) {
  if (i < a.D / 2) {
    const double rho = exp2(a.neg2_over_d_log2base * (double)i) * 0.15915494309189535;
    sRho[i] = two_floats(rho);
    sRho[kRho16 + i] = two_floats(rho * 65536.0 - floor(rho * 65536.0));
  }
}
// A position for the rotation: a whole float below 2^24; from there on 2^16 * p16 + p.
constexpr int32_t kNearPos = 1 << 24;
__device__ __forceinline__ bool is_far(int32_t pos) { return pos <= -kNearPos || pos >= kNearPos; }
struct RowPos { float p, p16; };
template <bool FAR>
__device__ __forceinline__ RowPos row_pos(int32_t pos) {
  const bool far = FAR && is_far(pos);
  return RowPos{(float)(far ? pos & 0xffff : pos), far ? (float)(pos >> 16) : 0.f};
}
// fraction (plus a small error term) of p * (hi + lo): the product p * hi is rounded, its error is exact in an FMA, and
// only the fraction of the rounded part matters, so the sum is good to about 1e-7 for a whole |p| < 2^24
__device__ __forceinline__ float turn_fraction(float p, float2 rho) {
#pragma clang fp contract(off)          // the rounded product and its error term must stay two operations
  const float t_hi = p * rho.x;
  const float t_lo = __builtin_fmaf(p, rho.y, __builtin_fmaf(p, rho.x, -t_hi));
  return __builtin_amdgcn_fractf(t_hi) + t_lo;
}
// (cos, sin) of pos * theta for one pair, the angle in turns.  FAR (a wave with a position from 2^24 on): plus the turns
// of p16 times the fraction of 2^16 frequencies, which are exactly 0 for the other positions.  One float product with
// the rest of the position in another was off by up to 4e-6 of a turn there; this stays at 2e-7.
template <bool FAR> struct Rho { float2 lo; __device__ Rho(const float2* t) : lo(*t) {} };
template <> struct Rho<true> { float2 lo, hi; __device__ Rho(const float2* t) : lo(*t), hi(t[kRho16]) {} };
template <bool FAR>
__device__ __forceinline__ void rotary_factor(int32_t pos, const Rho<FAR>& rho, float& c, float& sn) {
  const RowPos r = row_pos<FAR>(pos);
  float fr = turn_fraction(r.p, rho.lo);
  if constexpr (FAR) fr += turn_fraction(r.p16, rho.hi);
  c = __builtin_amdgcn_cosf(fr);
  sn = __builtin_amdgcn_sinf(fr);
}

typedef float float4v __attribute__((ext_vector_type(4)));

// Four consecutive columns of a row in the epilogue's LDS tile: columns 32 j + 8 q + 4 hf .. + 3 of row 32 i + l32.
// Chunk c (16 bytes) of row r sits in slot c ^ (r % 16): eight-byte pieces of 32 rows and 16-byte pieces of 4 whole
// rows both touch every bank once.
__device__ __forceinline__ u32x2* epi_piece(unsigned char* lds, int lane, int i, int j, int q) {
  const int r = 32 * i + (lane & 31), g = 8 * j + 2 * q + (lane >> 5);
  return reinterpret_cast<u32x2*>(lds + r * 256 + (((g >> 1) ^ (r & 15)) * 16) + (g & 1) * 8);
}
__device__ __forceinline__ void epi_put(unsigned char* lds, int lane, int i, int j, int q, bool zero, float4v o) {
  const u32x2 t = {cvt_pk_bf16(o[0], o[1]), cvt_pk_bf16(o[2], o[3])};
  *epi_piece(lds, lane, i, j, q) = zero ? u32x2{0u, 0u} : t;
}

// What the epilogue needs to know of this lane's rows, requested at the start of the kernel.
template <int TM>
struct EpiRows {
  int32_t pos[TM];
  bool zero[TM];                       // an index outside x produces a zero row
};
template <int TM, int EPI>
__device__ __forceinline__ void load_epi_rows(const QkvArgs& a, int64_t m0, int lane, EpiRows<TM>& rows) {
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t m = min(m0 + 32 * i + (lane & 31), a.M - 1);
    const int64_t idx = a.gather ? (int64_t)a.gather[m] : 0;
    rows.zero[i] = idx < 0 || idx >= a.x_rows;
    if (is_rope(EPI)) rows.pos[i] = a.pos[m];
  }
}

// a * c + b * s with one rounding of the second product (stated, so that every tile rounds alike)
__device__ __forceinline__ float turned(float a, float c, float b, float s) {
#pragma clang fp contract(off)
  return __builtin_fmaf(a, c, b * s);
}
// Rotation of the 128 columns held by a wave; the pair of a column is in the same lane.  JP: 32-column blocks of half
// a head (half-split pairs), or 0: interleaved pairs.
template <int TM, int JP, bool FAR>
__device__ __forceinline__ void epi_rotate(floatx16 (&acc)[TM][4], const float2* sRho, unsigned char* lds, int lane, int D,
                                           const EpiRows<TM>& rows) {
  const int hf = lane >> 5;
  if constexpr (JP > 0) {
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      const int j = JP == 2 ? jj : 2 * jj;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if constexpr (FAR) __builtin_amdgcn_sched_barrier(0);
        const float2* t = sRho + 32 * (j % JP) + 8 * q + 4 * hf;
        const Rho<FAR> rho[4] = {t, t + 1, t + 2, t + 3};
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          float4v o0, o1;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            float wx, wy;
            rotary_factor<FAR>(rows.pos[i], rho[c], wx, wy);
            const float f0 = acc[i][j][4 * q + c], f1 = acc[i][j + JP][4 * q + c];
            o0[c] = turned(f0, wx, -f1, wy);
            o1[c] = turned(f1, wx, f0, wy);
          }
          epi_put(lds, lane, i, j, q, rows.zero[i], o0);
          epi_put(lds, lane, i, j + JP, q, rows.zero[i], o1);
        }
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int p0 = (((32 * j) & (D - 1)) >> 1) + 4 * q + 2 * hf;
        if constexpr (FAR) __builtin_amdgcn_sched_barrier(0);
        const Rho<FAR> rho0(sRho + p0), rho1(sRho + p0 + 1);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          float wx, wy, vx, vy;
          rotary_factor<FAR>(rows.pos[i], rho0, wx, wy);
          rotary_factor<FAR>(rows.pos[i], rho1, vx, vy);
          const float f0 = acc[i][j][4 * q], f1 = acc[i][j][4 * q + 1], f2 = acc[i][j][4 * q + 2], f3 = acc[i][j][4 * q + 3];
          epi_put(lds, lane, i, j, q, rows.zero[i],
                  float4v{turned(f0, wx, -f1, wy), turned(f1, wx, f0, wy), turned(f2, vx, -f3, vy), turned(f3, vx, f2, vy)});
        }
      }
  }
}

// Epilogue of a wave that holds 32*TM rows x 128 columns of the product: acc[i][j] register v of a lane is row
// 32 i + lane%32, column 32 j + 8 (v / 4) + 4 (lane / 32) + v % 4 (weights as the A operand, activations as B).
// The rotary partner of a column, or the gate of an up column, is then in the same lane, and a lane needs the
// position of one row per 32.  The wave works alone in 32*TM * 256 bytes of LDS: residual rows come in through it
// with 16-byte loads, results are rounded to bf16 and leave through it with 16-byte stores.
// (With the tile going through LDS as fp32 for the whole workgroup, 128 columns at a time, a 256 x 256 tile spent
// about 20 us behind its last k-tile; now about 8.)
template <int TM, int EPI>
__device__ __forceinline__ void wave_epilogue(const QkvArgs& a, const OutTile& ot, floatx16 (&acc)[TM][4],
                                              const float2* sRho, unsigned char* lds, int64_t m0, int lane,
                                              const EpiRows<TM>& rows) {
  if constexpr (EPI == kAdd) {
    const int ch = lane & 15, rq = lane >> 4;
    const bf16_t* res = a.residual + ot.out_col0 + ch * 8;
#pragma unroll
    for (int b = 0; b < TM; ++b) {
      __builtin_amdgcn_sched_barrier(0);
      u32x4 t[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t m = min(m0 + 32 * b + 4 * u + rq, a.M - 1);      // (no branches while the accumulators are live)
        t[u] = *reinterpret_cast<const u32x4*>(res + m * ot.out_cols);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = 32 * b + 4 * u + rq;
        *reinterpret_cast<u32x4*>(lds + r * 256 + ((ch ^ (r & 15)) * 16)) = t[u];
      }
    }
  }
  if constexpr (EPI == kGlu) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float4v o;
#pragma unroll
          for (int c = 0; c < 4; ++c) {          // gate and up are rounded to bf16 first, as the separate calls store them
            const uint32_t gu = cvt_pk_bf16(acc[i][j][4 * q + c], acc[i][j + 2][4 * q + c]);
            o[c] = silu_mul(__uint_as_float(gu << 16), __uint_as_float(gu & 0xffff0000u));
          }
          epi_put(lds, lane, i, j, q, rows.zero[i], o);
        }
    const int ch = lane & 7, rq = lane >> 3;     // 64 columns: eight rows per store
    bf16_t* dst = ot.out + ot.out_col0 + ch * 8;
#pragma unroll
    for (int u = 0; u < 4 * TM; ++u) {
      const int r = 8 * u + rq;
      const int64_t m = m0 + r;
      if (m < a.M) *reinterpret_cast<u32x4*>(dst + m * ot.out_cols) = *reinterpret_cast<const u32x4*>(lds + r * 256 + ((ch ^ (r & 15)) * 16));
    }
    return;
  }
  bool rotated = false;
  if constexpr (is_rope(EPI)) {
    if (ot.rotate) {
      constexpr int JP = EPI == kRopeHalf128 ? 2 : EPI == kRopeHalf64 ? 1 : 0;
      bool far = false;
#pragma unroll
      for (int i = 0; i < TM; ++i) far |= is_far(rows.pos[i]);
      if (__builtin_expect(__any(far), 0)) epi_rotate<TM, JP, true>(acc, sRho, lds, lane, a.D, rows);
      else epi_rotate<TM, JP, false>(acc, sRho, lds, lane, a.D, rows);
      rotated = true;
    }
  }
  if (!rotated) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        __builtin_amdgcn_sched_barrier(0);       // (else every LDS read of the residual is hoisted, and spilled)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float4v o = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          if constexpr (EPI == kAdd) {
            const u32x2 t = *epi_piece(lds, lane, i, j, q);
            o[0] += __uint_as_float(t.x << 16); o[1] += __uint_as_float(t.x & 0xffff0000u);
            o[2] += __uint_as_float(t.y << 16); o[3] += __uint_as_float(t.y & 0xffff0000u);
          }
          epi_put(lds, lane, i, j, q, rows.zero[i], o);
        }
      }
  }
  const int ch = lane & 15, rq = lane >> 4;
  bf16_t* dst = ot.out + ot.out_col0 + ch * 8;
  bf16_t* fus = ot.fused + ot.out_col0 + ch * 8;
#pragma unroll
  for (int b = 0; b < TM; ++b) {
    int32_t d[8];                      // (requested together, before the first store waits for one)
    if (is_rope(EPI) && ot.fused) {
#pragma unroll
      for (int u = 0; u < 8; ++u) d[u] = a.dst_rows[min(m0 + 32 * b + 4 * u + rq, a.M - 1)];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int r = 32 * b + 4 * u + rq;
      const int64_t m = m0 + r;
      if (m < a.M) {
        const u32x4 t = *reinterpret_cast<const u32x4*>(lds + r * 256 + ((ch ^ (r & 15)) * 16));
        *reinterpret_cast<u32x4*>(dst + m * ot.out_cols) = t;
        if (is_rope(EPI) && ot.fused && d[u] >= 0 && d[u] < a.fused_rows)
          *reinterpret_cast<u32x4*>(fus + (int64_t)d[u] * ot.out_cols) = t;
      }
    }
  }
}

// Staged tiles have rows of 128 bytes (8 chunks of 16 bytes) without padding; chunk c of row r sits in
// slot c ^ ((r / 2) % 8), so the 16-byte fragment reads of 16 consecutive rows touch 16 different bank
// groups.  One load instruction of a wave fills 8 rows (1 KB): lane L fills slot L%8 of row L/8.

// ---- load/compute-split kernel: 32*TM*NC-row tiles x 128 columns ---------------------------------------
// NC compute waves (32*TM x 128 outputs each) issue only fragment reads and MFMAs; four more waves only issue the
// asynchronous global-to-LDS loads.  A wave that issues such a load can stall on the memory pipeline's queue, and a
// stalled wave issues no MFMAs either: with the two roles in different waves the matrix unit keeps running meanwhile.
// S stages: S - 1 k-tiles are on their way while one is used (the deeper rings belong to the small tiles, whose
// launches stream the weights from HBM: 64 x 128 tiles keep 120 KB in flight per compute unit).
//
// Synchronisation, one barrier per k-tile (barrier number kt + 1 is crossed while tile kt is computed):
//   compute wave: steps 0..2 of tile kt, wait for its last fragment reads of stage kt%S, barrier,
//                 request the first fragments of tile kt+1, step 3 of tile kt;
//   load wave:    after barrier kt it requests tile kt+S-1 into stage (kt+S-1)%S == (kt-1)%S (free: every
//                 compute wave finished reading tile kt-1 before barrier kt), waits until its loads of
//                 tile kt+1 have landed, barrier.
template <int TM_, int NC_, int S_>
struct WsTile {
  static constexpr int TM = TM_, TN = 4, NC = NC_, NL = 4, S = S_;
  static constexpr int BM = 32 * TM * NC;
  static constexpr int NTHR = 64 * (NC + NL);
  static constexpr int A_LD = BM / 8 / NL;                        // 1 KB load instructions per load wave and stage
  static constexpr int B_LD = kBN / 8 / NL;
  static constexpr int STAGE = (BM + kBN) * kBK * 2;
  static constexpr size_t LDS_MAIN = (size_t)S * STAGE;
  static constexpr size_t LDS = LDS_MAIN + kRhoBytes;
  static_assert(32 * TN == kBN, "a compute wave covers the 128 output columns");
  static_assert(NC * TM * 8192 <= (int)LDS_MAIN, "the epilogue works in the ring");
};

// Re-rotation of rows r0 .. r0 + n - 1 of the cache (at most kSideRows) by one workgroup.  Their chunks, the rows that the product writes and the
// (cos, sin) pairs are worked out in LDS, then every thread keeps four pieces of keys and values on their way (two vectors of
// each, the halves of eight rotary pairs).  64 compute units re-rotate 8192 rows of 8 heads beside a product of 192 workgroups
// that takes 32.3 us alone and 33.5 so; the launch of its own took 13.9.
struct SideLds {
  qcf_chunk table[kSideChunks];
  int16_t chunk[kSideRows];                       // of a row; -1: none, or a row of the product
  int first, last;                                // chunks of the first and the last row
  float2 cs[(kSideRows + 1) * 64];
};
template <int NTHR>
__device__ __forceinline__ void rerope_rows(const QkvArgs& a, int64_t r0, int n, unsigned char* smem) {
  SideLds& l = *reinterpret_cast<SideLds*>(smem);
  const SideRerope& s = a.side;
  const int tid = threadIdx.x, half = a.D / 2;
  for (int i = tid; i < s.n_chunks * (int)(sizeof(qcf_chunk) / 8); i += NTHR)
    reinterpret_cast<uint64_t*>(l.table)[i] = reinterpret_cast<const uint64_t*>(s.chunks)[i];
  __syncthreads();
  for (int i = tid; i < n; i += NTHR) {
    const int c = chunk_of(l.table, s.n_chunks, r0 + i);
    const qcf_chunk& ch = l.table[c];
    l.chunk[i] = r0 + i >= ch.dst_row && r0 + i < ch.dst_row + ch.len ? (int16_t)c : (int16_t)-1;
    if (i == 0) l.first = c;
    if (i == n - 1) l.last = c;
  }
  __syncthreads();
  for (int64_t i = tid; i < a.M; i += NTHR) {
    const int64_t row = (int64_t)a.dst_rows[i] - r0;
    if (row >= 0 && row < n) l.chunk[row] = -1;
  }
  // (at most one chunk more than rows where each has a token; rows of what a table of empty chunks has beyond are left as they are)
  const int first = l.first, pairs = min(l.last - first + 1, kSideRows + 1) * half;
  for (int i = tid; i < pairs; i += NTHR) {
    l.cs[i] = shift_pair(l.table[first + i / half], a.neg2_over_d_log2base, i % half);
  }
  __syncthreads();
  const int row_elems = a.Hkv * a.D, per_head = half / 8, slots = a.Hkv * per_head, items = n * slots;
  constexpr int U = 4;
  for (int i0 = tid; i0 < items; i0 += U * NTHR) {
    u32x4 k[U][2], v[U][2];
    int at[U], c[U], e0[U], e1[U], p0[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * NTHR;
      at[u] = min(i, items - 1) / slots;
      const int slot = min(i, items - 1) - at[u] * slots, head = slot / per_head;
      p0[u] = (slot - head * per_head) * 8;
      e0[u] = head * a.D + (s.style == 0 ? p0[u] : 2 * p0[u]);
      e1[u] = e0[u] + (s.style == 0 ? half : 8);
      c[u] = i < items ? l.chunk[at[u]] : -1;
      if ((c[u] - first) * half >= pairs) c[u] = -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c[u] >= 0) {
        const qcf_chunk& ch = l.table[c[u]];
        const int64_t off = (r0 + at[u] - ch.dst_row) * row_elems;
        const bf16_t* ks = static_cast<const bf16_t*>(ch.k_src) + off;
        const bf16_t* vs = static_cast<const bf16_t*>(ch.v_src) + off;
        k[u][0] = *reinterpret_cast<const u32x4*>(ks + e0[u]);
        k[u][1] = *reinterpret_cast<const u32x4*>(ks + e1[u]);
        v[u][0] = *reinterpret_cast<const u32x4*>(vs + e0[u]);
        v[u][1] = *reinterpret_cast<const u32x4*>(vs + e1[u]);
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (c[u] >= 0) {
        float f[16], o[16];
        Vec16<bf16_t>::unpack(k[u][0], f);
        Vec16<bf16_t>::unpack(k[u][1], f + 8);
        const float2* cs = l.cs + (c[u] - first) * half + p0[u];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (s.style == 0) turn_pair(f[e], f[e + 8], cs[e], o[e], o[e + 8]);
          else turn_pair(f[2 * e], f[2 * e + 1], cs[e], o[2 * e], o[2 * e + 1]);
        }
        const int64_t dst = (r0 + at[u]) * row_elems;
        *reinterpret_cast<u32x4*>(a.k_fused + dst + e0[u]) = mk4(cvt_pk_bf16(o[0], o[1]), cvt_pk_bf16(o[2], o[3]), cvt_pk_bf16(o[4], o[5]), cvt_pk_bf16(o[6], o[7]));
        *reinterpret_cast<u32x4*>(a.k_fused + dst + e1[u]) = mk4(cvt_pk_bf16(o[8], o[9]), cvt_pk_bf16(o[10], o[11]), cvt_pk_bf16(o[12], o[13]), cvt_pk_bf16(o[14], o[15]));
        *reinterpret_cast<u32x4*>(a.v_fused + dst + e0[u]) = v[u][0];
        *reinterpret_cast<u32x4*>(a.v_fused + dst + e1[u]) = v[u][1];
      }
  }
}

// WIDE: x is 4 GiB or larger (64-bit addresses per lane instead of 32-bit offsets)
template <typename C, int EPI, bool WIDE>
__global__ __launch_bounds__(C::NTHR) void qkv_ws_kernel(QkvArgs a) {
  static_assert(sizeof(SideLds) <= C::LDS_MAIN, "the re-rotation works in the ring");
  constexpr int TM = C::TM, TN = C::TN, S = C::S;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hf = lane >> 5, l32 = lane & 31;
  if constexpr (is_rope(EPI)) {
    if ((int)blockIdx.x >= a.side.first_wg) {
      const int64_t r0 = ((int)blockIdx.x - a.side.first_wg) * (int64_t)a.side.rows, r1 = min(r0 + a.side.rows, a.side.total_rows);
      for (int64_t r = r0; r < r1; r += kSideRows) {
        rerope_rows<C::NTHR>(a, r, (int)min((int64_t)kSideRows, r1 - r), smem);
        __syncthreads();
      }
      return;
    }
  }
  // consecutive workgroup ids land on different XCDs: all row tiles of a (column block, contraction range) share an
  // XCD, so its weights are fetched into one L2 only
  const int units = a.n_tiles * a.splits;
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  int m_tile = slot % a.m_tiles, unit = (slot / a.m_tiles) * 8 + xcd;
  if (a.rows_over_xcds) {          // many row tiles: row tiles are dealt to the XCDs, column tiles run side by side
    m_tile = (slot / units) * 8 + xcd;
    unit = slot % units;
  }
  if (unit >= units || m_tile >= a.m_tiles) return;
  const int split = unit / a.n_tiles, n_tile = unit - split * a.n_tiles;
  const int64_t m0 = (int64_t)m_tile * C::BM;
  const int block = a.n_tile0 + n_tile;
  const OutTile ot = out_tile_of<EPI>(a, block);
  if (!ot.out) return;
  const int kt0 = split * a.split_len;
  const int nk = min(a.d_model / kBK - kt0, a.split_len);
  float2* sRho = reinterpret_cast<float2*>(smem + C::LDS_MAIN);

  if (wave >= C::NC) {
    // ---------------- load wave lw: instruction i covers tile rows 8*(lw + NL*i) .. +7
    const int lw = wave - C::NC;
    const int ld_r = lane >> 3;
    const uint32_t row_bytes = (uint32_t)a.d_model * 2u;
    uint32_t a_off[WIDE ? 1 : C::A_LD];                          // byte offset from x
    const char* a_ptr[WIDE ? C::A_LD : 1];
    const char* a_base = reinterpret_cast<const char*>(a.x) + (int64_t)kt0 * kBK * 2;
#pragma unroll
    for (int i = 0; i < C::A_LD; ++i) {
      const int row = 8 * (lw + C::NL * i) + ld_r;
      const int chunk = (lane & 7) ^ ((row >> 1) & 7);
      const int64_t m = m0 + row;
      int64_t idx = 0;                                           // rows past M read row 0; never stored
      if (m < a.M) {
        idx = a.gather ? (int64_t)a.gather[m] : m;
        if (idx < 0 || idx >= a.x_rows) idx = 0;                 // stored as zeros in the epilogue
      }
      if constexpr (WIDE) a_ptr[i] = a_base + idx * (int64_t)row_bytes + chunk * 16;
      else a_off[i] = (uint32_t)idx * row_bytes + (uint32_t)chunk * 16u;
    }
    uint32_t b_off[C::B_LD];
#pragma unroll
    for (int i = 0; i < C::B_LD; ++i) {
      const int row = 8 * (lw + C::NL * i) + ld_r;
      const int chunk = (lane & 7) ^ ((row >> 1) & 7);
      b_off[i] = block_w_step<EPI>(a, row) * row_bytes + (uint32_t)chunk * 16u;
    }
    const char* b_base = reinterpret_cast<const char*>(a.w + block_w_row<EPI>(block) * a.d_model) + (int64_t)kt0 * kBK * 2;
    auto issue = [&](int kt) {
      unsigned char* sA = smem + (size_t)(kt % S) * C::STAGE;
      unsigned char* sB = sA + C::BM * kBK * 2;
#pragma unroll
      for (int i = 0; i < C::B_LD; ++i)
        load_to_lds(b_base + (int64_t)kt * kBK * 2, b_off[i], sB + (lw + C::NL * i) * 1024);
#pragma unroll
      for (int i = 0; i < C::A_LD; ++i) {
        if constexpr (WIDE) load_to_lds_addr(a_ptr[i] + (int64_t)kt * kBK * 2, sA + (lw + C::NL * i) * 1024);
        else load_to_lds(a_base + (int64_t)kt * kBK * 2, a_off[i], sA + (lw + C::NL * i) * 1024);
      }
    };
    constexpr int kFlight = (S - 2) * (C::A_LD + C::B_LD);       // loads that may stay on their way: all but the next tile's
    static_assert(kFlight <= 63, "the wait counter holds 6 bits");
    for (int kt = 0; kt < min(S - 1, nk); ++kt) issue(kt);
    if (nk >= S - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kFlight) : "memory");
    else __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();                                             // barrier 0: tile 0 has landed
    for (int kt = 0; kt < nk; ++kt) {
      if (kt + S - 1 < nk) {
        issue(kt + S - 1);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kFlight) : "memory");
      } else {
        __builtin_amdgcn_s_waitcnt(0);
      }
      __syncthreads();                                           // barrier kt + 1: tile kt + 1 has landed
    }
    if (is_rope(EPI) && lw == 0) fill_rho(a, sRho, lane);           // (behind the ring: no stage is touched)
    __syncthreads();                                             // the ring is free, the frequencies are there
  } else {
    // ---------------- compute wave: rows 32*TM*wave .. of the tile, all 128 columns
    __builtin_amdgcn_s_setprio(2);                               // its instructions go first when both roles are ready
    const int swz = (l32 >> 1) & 7;
    const int fb0 = l32 * 128 + ((hf ^ (swz & 1)) * 16) + ((swz & 6) * 16);
    const int a_frag = wave * 32 * TM * 128 + fb0;
    const int b_frag = C::BM * kBK * 2 + fb0;
    EpiRows<TM> rows;
    load_epi_rows<TM, EPI>(a, m0 + wave * 32 * TM, lane, rows);
    floatx16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = floatx16{0};
    u32x4 af[2][TM], bfr[2][TN];
    auto fetch = [&](const unsigned char* stage, int ks, int buf) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
        af[buf][i] = *reinterpret_cast<const u32x4*>(stage + ((a_frag + i * 32 * 128) ^ (32 * ks)));
#pragma unroll
      for (int j = 0; j < TN; ++j)
        bfr[buf][j] = *reinterpret_cast<const u32x4*>(stage + ((b_frag + j * 32 * 128) ^ (32 * ks)));
    };
    auto mfmas = [&](int buf) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bfr[buf][j]),
                                                               __builtin_bit_cast(bf16x8, af[buf][i]), acc[i][j], 0, 0, 0);
    };
    // issue order of one k-step: every fragment read sits behind an MFMA, so that the matrix unit is
    // already busy while the read is issued
    auto interleave = [&]() {
      constexpr int kPairs = TM * TN < TM + TN ? TM * TN : TM + TN;
#pragma unroll
      for (int q = 0; q < kPairs; ++q) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // one MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);       // one LDS read
      }
      if (TM * TN > kPairs) __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - kPairs, 0);
      if (TM + TN > kPairs) __builtin_amdgcn_sched_group_barrier(0x100, TM + TN - kPairs, 0);
    };
    __syncthreads();                                             // barrier 0
    fetch(smem, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
      const unsigned char* stage = smem + (size_t)(kt % S) * C::STAGE;
#pragma unroll
      for (int ks = 0; ks < 3; ++ks) {
        fetch(stage, ks + 1, (ks + 1) & 1);
        mfmas(ks & 1);
        interleave();
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");         // the last fragments of this stage are in registers
      __syncthreads();                                           // barrier kt + 1
      // (after the last tile this re-reads the current stage; the values are not used)
      fetch(smem + (size_t)((kt + 1 < nk ? kt + 1 : kt) % S) * C::STAGE, 0, 0);
      mfmas(1);
      interleave();
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    if (a.splits > 1) {
      if constexpr (TM == 1) {        // partial sums in register order: 1 KB per store
        float4* dst = static_cast<float4*>(a.part) + ((((int64_t)split * a.n_tiles + n_tile) * a.m_tiles + m_tile) * C::NC + wave) * 1024 + lane;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            dst[(4 * j + q) * 64] = make_float4(acc[0][j][4 * q], acc[0][j][4 * q + 1], acc[0][j][4 * q + 2], acc[0][j][4 * q + 3]);
      }
      return;
    }
    wave_epilogue<TM, EPI>(a, ot, acc, sRho, smem + wave * TM * 8192, m0 + wave * 32 * TM, lane, rows);
  }
}

// Sums the partial results of a split contraction, in range order, and finishes them.  One workgroup per 32 rows x 64 columns of a
// block: the two 32-column parts that hold the halves of rotary pairs, gate and up, or else neighbours, so that a thread
// has both partners of its eight sums and finishes them itself; the results pass through LDS to leave as 16-byte pieces.  Bound by
// latency where rows are few: launch, one round of loads, stores.  (128 columns to a workgroup, finished by its first wave alone:
// calls of 61 rows, K 4096, N 4096 in six ranges 15.4 us, now 14.5; 100 rows, K 4096, N 6144 in four 20.3 and 19.7; 200 rows 26.6
// and 26.0.)
template <int EPI>
__global__ __launch_bounds__(256) void qkv_split_reduce(QkvArgs a, int n_groups) {
  constexpr int LD = 68;                                         // floats of a row (an odd number of 16-byte pieces)
  constexpr bool kApart = EPI == kRopeHalf128 || EPI == kGlu;    // the parts are 64 columns apart
  constexpr int kChunks = EPI == kGlu ? 4 : 8;                   // 16-byte pieces of a result row
  __shared__ __align__(16) float sOut[32 * LD];
  __shared__ float2 sRho[2 * kRho16];
  const int tid = threadIdx.x, lane = tid & 63, q = tid >> 6, hf = lane >> 5;
  const int grp = blockIdx.x, n_tile = blockIdx.y, half = blockIdx.z;
  const OutTile ot = out_tile_of<EPI>(a, a.n_tile0 + n_tile);
  if (!ot.out) return;
  const int j0 = kApart ? half : 2 * half, j1 = kApart ? half + 2 : 2 * half + 1;
  const int64_t m0 = (int64_t)grp * 32;
  // the piece that this thread stores: row sr, eight columns from sc on (of the block's)
  const int sr = tid / kChunks, chunk = tid % kChunks;
  const int sc = kApart ? (chunk < 4 ? 32 * j0 + 8 * chunk : 32 * j1 + 8 * (chunk - 4)) : 64 * half + 8 * chunk;
  const bool stores = sr < 32 && m0 + sr < a.M;
  EpiRows<1> rows;
  load_epi_rows<1, EPI>(a, m0, lane, rows);
  u32x4 res{};
  int32_t fused_row = -1;
  if (stores) {
    if (EPI == kAdd) res = *reinterpret_cast<const u32x4*>(a.residual + (m0 + sr) * ot.out_cols + ot.out_col0 + sc);
    if (is_rope(EPI) && ot.fused) fused_row = a.dst_rows[m0 + sr];
  }
  const float4* src = static_cast<const float4*>(a.part) + ((int64_t)n_tile * n_groups + grp) * 1024 + lane;
  const int at0 = (4 * j0 + q) * 64, at1 = (4 * j1 + q) * 64;
  const int64_t stride = (int64_t)a.n_tiles * n_groups * 1024;
  float4 s0 = src[at0], s1 = src[at1];
  // ranges that are on their way together: four, then two, then one (one after the other they cost 0.3 us each)
  auto add = [&](auto n_c) {
    constexpr int N = decltype(n_c)::value;
    float4 t[N][2];
#pragma unroll
    for (int u = 0; u < N; ++u) { t[u][0] = src[(u + 1) * stride + at0]; t[u][1] = src[(u + 1) * stride + at1]; }
    src += N * stride;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      s0.x += t[u][0].x; s0.y += t[u][0].y; s0.z += t[u][0].z; s0.w += t[u][0].w;
      s1.x += t[u][1].x; s1.y += t[u][1].y; s1.z += t[u][1].z; s1.w += t[u][1].w;
    }
  };
  int left = a.splits - 1;
  for (; left >= 4; left -= 4) add(std::integral_constant<int, 4>{});
  if (left & 2) add(std::integral_constant<int, 2>{});
  if (left & 1) add(std::integral_constant<int, 1>{});
  float f0[4] = {s0.x, s0.y, s0.z, s0.w}, f1[4] = {s1.x, s1.y, s1.z, s1.w};      // columns 32 j + 8 q + 4 hf .. + 3 of row lane % 32
  if constexpr (is_rope(EPI)) {
    if (tid < 64) fill_rho(a, sRho, tid);
    __syncthreads();
    auto rotate = [&](auto far_c) {
      constexpr bool FAR = decltype(far_c)::value;
      if constexpr (EPI == kRopeInter) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          float(&f)[4] = i == 0 ? f0 : f1;
          const float2* t = sRho + ((32 * (i == 0 ? j0 : j1) & (a.D - 1)) >> 1) + 4 * q + 2 * hf;
#pragma unroll
          for (int c = 0; c < 2; ++c) {
            float wx, wy;
            rotary_factor<FAR>(rows.pos[0], Rho<FAR>(t + c), wx, wy);
            const float x = f[2 * c], y = f[2 * c + 1];
            f[2 * c] = turned(x, wx, -y, wy);
            f[2 * c + 1] = turned(y, wx, x, wy);
          }
        }
      } else {
        const float2* t = sRho + (EPI == kRopeHalf128 ? 32 * half : 0) + 8 * q + 4 * hf;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float wx, wy;
          rotary_factor<FAR>(rows.pos[0], Rho<FAR>(t + c), wx, wy);
          const float x = f0[c], y = f1[c];
          f0[c] = turned(x, wx, -y, wy);
          f1[c] = turned(y, wx, x, wy);
        }
      }
    };
    if (ot.rotate) {
      if (__builtin_expect(__any(is_far(rows.pos[0])), 0)) rotate(std::true_type{});
      else rotate(std::false_type{});
    }
  }
  if constexpr (EPI == kGlu) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {                // gate and up are rounded to bf16 first, as the separate calls store them
      const uint32_t gu = cvt_pk_bf16(f0[c], f1[c]);
      f0[c] = silu_mul(__uint_as_float(gu << 16), __uint_as_float(gu & 0xffff0000u));
    }
  }
  if (rows.zero[0]) {
#pragma unroll
    for (int c = 0; c < 4; ++c) f0[c] = f1[c] = 0.f;
  }
  float* mine = sOut + (lane & 31) * LD + 8 * q + 4 * hf;
  *reinterpret_cast<float4*>(mine) = make_float4(f0[0], f0[1], f0[2], f0[3]);
  if (EPI != kGlu) *reinterpret_cast<float4*>(mine + 32) = make_float4(f1[0], f1[1], f1[2], f1[3]);
  __syncthreads();
  if (!stores) return;
  const float4 o0 = *reinterpret_cast<const float4*>(sOut + sr * LD + 8 * chunk), o1 = *reinterpret_cast<const float4*>(sOut + sr * LD + 8 * chunk + 4);
  float o[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
  if (EPI == kAdd) {
    const uint32_t r[4] = {res.x, res.y, res.z, res.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) { o[2 * c] += __uint_as_float(r[c] << 16); o[2 * c + 1] += __uint_as_float(r[c] & 0xffff0000u); }
  }
  const u32x4 t = mk4(cvt_pk_bf16(o[0], o[1]), cvt_pk_bf16(o[2], o[3]), cvt_pk_bf16(o[4], o[5]), cvt_pk_bf16(o[6], o[7]));
  *reinterpret_cast<u32x4*>(ot.out + (m0 + sr) * ot.out_cols + ot.out_col0 + sc) = t;
  if (is_rope(EPI) && ot.fused && fused_row >= 0 && fused_row < a.fused_rows)
    *reinterpret_cast<u32x4*>(ot.fused + (int64_t)fused_row * ot.out_cols + ot.out_col0 + sc) = t;
}

// ---- 256 x 256 tiles, four waves of 128 x 128 -----------------------------------------------------
// One wave per SIMD, so that a wave can hold 128 x 128 outputs (256 accumulation registers) and an LDS fragment
// feeds four MFMAs.  Both operands of a k-tile are kept as two units of 128 rows (the rows 64 u .. 64 u + 63 of both
// wave rows / wave columns), and a k-tile runs as four phases of 16 MFMAs over the operand halves
//     phase 0: A0 x B0     phase 1: A0 x B1     phase 2: A1 x B1     phase 3: A1 x B0
// with the fragments of a half (two 32-row blocks, four k-steps) in registers.  Phase p reads the half that phase
// p + 1 adds - B1(t), A1(t), A0(t+1), B0(t+1) - so every unit is read in one phase only and its LDS can be refilled
// right behind it: the loads of a unit have seven phases (about 2 us) to arrive although the ring holds just two
// k-tiles.  One barrier per phase publishes the unit that the next phase reads and frees the one this phase read.
// 1024 x 1024 blocks of workgroups keep to an XCD (locate_big_tile).  Measured at M 23891, K 4096, N 6144: 870 us,
// 1.38 PFLOP/s (256 x 128 tiles: 1080 us); the clock settles at 1.75 GHz under this load, the matrix unit is busy
// 80 % of the cycles of the k-loop.
struct QuadTile {
  static constexpr int BM = 256, BN = 256, NTHR = 256;
  static constexpr int UNIT = 128 * kBK * 2;                       // 16 KB: 128 rows of one operand
  static constexpr int STAGE = 4 * UNIT;                           // A0 A1 B0 B1
  static constexpr size_t LDS = 2 * STAGE + kRhoBytes;
};

// End of a phase: this wave's fragment reads are back and at most N of its loads are still on their way.
template <int N>
__device__ __forceinline__ void wait_and_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (N >= 0) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
  else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Tile order: workgroups with the same id modulo 8 share an XCD and its 32 compute units run 32 of them at a time.
// Tiles are numbered row first inside groups of m_group row tiles, and each XCD takes 32 consecutive ones, i.e. a
// roughly square block whose operands fit its L2; the last, incomplete round is dealt out evenly.
__device__ __forceinline__ bool locate_big_tile(int m_tiles, int n_bt, int gm, int id, int& m_tile, int& b_tile) {
  const int total = m_tiles * n_bt;
  const int xcd = id & 7, slot = id >> 3;
  const int full = total / 256;
  int p;
  if (slot < 32 * full) {
    p = (slot >> 5) * 256 + xcd * 32 + (slot & 31);
  } else {
    const int q = (total - full * 256 + 7) >> 3, i = slot - 32 * full;
    if (i >= q) return false;
    p = full * 256 + xcd * q + i;
  }
  if (p >= total) return false;
  const int per_group = gm * n_bt;
  const int grp = p / per_group, r = p - grp * per_group;
  const int rows = min(gm, m_tiles - grp * gm);
  b_tile = r / rows;
  m_tile = grp * gm + (r - b_tile * rows);
  return true;
}

// SPLIT: column tiles are numbered once per range of the contraction, and the tile's sums leave as they are for
// qkv_split_reduce, straight from the accumulators (a template parameter, so that the whole product's registers stay)
template <int EPI, bool SPLIT>
__global__ __launch_bounds__(256, 1) void qkv_quad_kernel(QkvArgs a) {
  using C = QuadTile;
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int hf = lane >> 5, l32 = lane & 31;
  const int n_bt = (a.n_tiles + 1) / 2;
  int m_tile, b_tile;
  if (!locate_big_tile(a.m_tiles, SPLIT ? n_bt * a.splits : n_bt, a.m_group, (int)blockIdx.x, m_tile, b_tile)) return;
  int split = 0, nk = a.d_model / kBK;                           // even (launcher)
  if constexpr (SPLIT) {
    split = b_tile / n_bt;
    b_tile -= split * n_bt;
    nk = min(nk - split * a.split_len, a.split_len);             // even as well: split_len is
  }
  const int64_t k0 = SPLIT ? (int64_t)split * a.split_len * (kBK * 2) : 0;       // bytes of a row in front of the range
  const int64_t m0 = (int64_t)m_tile * C::BM;
  const int block0 = a.n_tile0 + 2 * b_tile;
  const bool second = 2 * b_tile + 1 < a.n_tiles;                // (else the tile's second 128 columns repeat the first)
  const uint32_t row_bytes = (uint32_t)a.d_model * 2u;

  // byte offsets of this lane's 16 bytes inside k-tile 0: load i of unit u fills unit rows 8*wave + 32*i .. +7
  uint32_t a_off[2][4], b_off[2][4];
  {
    const int ld_r = lane >> 3;
    const uint32_t chunk = (uint32_t)(((lane & 7) ^ ((4 * wave + (ld_r >> 1)) & 7)) * 16);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = u * 64 + (i & 1) * 32 + 8 * wave + ld_r;
        const int64_t m = m0 + (i >> 1) * 128 + r;
        int64_t idx = 0;                                         // rows past M read row 0; never stored
        if (m < a.M) {
          idx = a.gather ? (int64_t)a.gather[m] : m;
          if (idx < 0 || idx >= a.x_rows) idx = 0;               // stored as zeros in the epilogue
        }
        a_off[u][i] = (uint32_t)idx * row_bytes + chunk;
        const uint32_t blk_rows = second && i >= 2 ? (uint32_t)block_w_row<EPI>(1) : 0u;
        b_off[u][i] = (blk_rows + block_w_step<EPI>(a, r)) * row_bytes + chunk;
      }
  }
  const uint32_t lds0 = lds_offset_of(smem);
  const uint32_t lds_w = __builtin_amdgcn_readfirstlane((int)(lds0 + (uint32_t)wave * 1024u));
  const char* a_base = reinterpret_cast<const char*>(a.x) + k0;
  const char* b_base = reinterpret_cast<const char*>(a.w + block_w_row<EPI>(block0) * a.d_model) + k0;
  auto load_a1 = [&](auto u_c, auto i_c, auto sl_c, const char* src) {
    constexpr int u = decltype(u_c)::value, i = decltype(i_c)::value, sl = decltype(sl_c)::value;
    load_to_lds_const<sl * C::STAGE + u * C::UNIT + i * 4096>(src, a_off[u][i], lds_w);
  };
  auto load_b1 = [&](auto u_c, auto i_c, auto sl_c, const char* src) {
    constexpr int u = decltype(u_c)::value, i = decltype(i_c)::value, sl = decltype(sl_c)::value;
    load_to_lds_const<sl * C::STAGE + (2 + u) * C::UNIT + i * 4096>(src, b_off[u][i], lds_w);
  };
  std::integral_constant<int, 0> c0;
  std::integral_constant<int, 1> c1;
  std::integral_constant<int, 2> c2;
  std::integral_constant<int, 3> c3;
  // (the last tiles load the last k-tile again, into slots that nothing reads any more: one loop body for all tiles)
  auto k_off = [&](int t) { return (int64_t)min(t, nk - 1) * (kBK * 2); };
  auto load_a = [&](auto u, auto sl, int t) {
    const char* p = a_base + k_off(t);
    load_a1(u, c0, sl, p); load_a1(u, c1, sl, p); load_a1(u, c2, sl, p); load_a1(u, c3, sl, p);
  };
  auto load_b = [&](auto u, auto sl, int t) {
    const char* p = b_base + k_off(t);
    load_b1(u, c0, sl, p); load_b1(u, c1, sl, p); load_b1(u, c2, sl, p); load_b1(u, c3, sl, p);
  };

  const int swz = (l32 >> 1) & 7;
  const uint32_t fb0 = l32 * 128 + ((hf ^ (swz & 1)) * 16) + ((swz & 6) * 16);
  uint32_t fa[2][4], fb[2][4];                                   // fragment addresses: [slot][k-step], half 0
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      fa[s][ks] = lds0 + s * C::STAGE + wm * 8192 + (fb0 ^ (32 * ks));
      fb[s][ks] = lds0 + s * C::STAGE + 2 * C::UNIT + wn * 8192 + (fb0 ^ (32 * ks));
    }
  auto lds16 = [](uint32_t addr) { return *(const u32x4 __attribute__((address_space(3)))*)(uintptr_t)addr; };

  EpiRows<4> rows;
  if constexpr (!SPLIT) load_epi_rows<4, EPI>(a, m0 + wm * 128, lane, rows);
  floatx16 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx16{0};
  u32x4 ra[2][2][4], rb[2][2][4];      // [register set][32-row block][k-step]; B half u of tile t is in set u ^ (t & 1)

  load_a(c0, c0, 0); load_b(c0, c0, 0); load_b(c1, c0, 0); load_a(c1, c0, 0);
  load_a(c0, c1, 1); load_b(c0, c1, 1); load_b(c1, c1, 1); load_a(c1, c1, 1);
  wait_and_barrier<24>();              // A0(0) and B0(0) have landed
#pragma unroll
  for (int ii = 0; ii < 2; ++ii)
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      ra[0][ii][ks] = lds16(fa[0][ks] + ii * 4096);
      rb[0][ii][ks] = lds16(fb[0][ks] + ii * 4096);
    }
  wait_and_barrier<-1>();
  load_a(c0, c0, 2);
  wait_and_barrier<24>();              // B1(0) has landed

  auto phase = [&](auto par_c, auto ph_c, const char* src) {
    constexpr int PAR = decltype(par_c)::value, ph = decltype(ph_c)::value;
    std::integral_constant<int, PAR> sl;
    std::integral_constant<int, PAR ^ 1> sln;
    constexpr int UA = ph >= 2 ? 1 : 0, UB = (ph == 1 || ph == 2) ? 1 : 0;      // operand halves of this phase
    auto rd = [&](auto n_c) {                                    // fragments for the next phase
      constexpr int n = decltype(n_c)::value, ks = n >> 1, ii = n & 1;
      if (ph == 0) rb[1 ^ PAR][ii][ks] = lds16(fb[PAR][ks] + C::UNIT + ii * 4096);           // B1(t)
      if (ph == 1) ra[1][ii][ks] = lds16(fa[PAR][ks] + C::UNIT + ii * 4096);                 // A1(t)
      if (ph == 2) ra[0][ii][ks] = lds16(fa[PAR ^ 1][ks] + ii * 4096);                       // A0(t+1)
      if (ph == 3) rb[1 ^ PAR][ii][ks] = lds16(fb[PAR ^ 1][ks] + ii * 4096);                 // B0(t+1)
    };
    auto load1 = [&](auto i) {                                   // refill of the unit the previous phase read
      if (ph == 0) load_b1(c0, i, sl, src);                      // B0(t+2)
      if (ph == 1) load_b1(c1, i, sl, src);                      // B1(t+2)
      if (ph == 2) load_a1(c1, i, sl, src);                      // A1(t+2)
      if (ph == 3) load_a1(c0, i, sln, src);                     // A0(t+3)
    };
    auto step = [&](auto n_c) {                                  // issue order: an LDS read or a load behind each MFMA
      constexpr int n = decltype(n_c)::value, ks = n >> 2, j = (n >> 1) & 1, i = (n & 1) ^ j;
      acc[2 * UA + i][2 * UB + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          __builtin_bit_cast(bf16x8, rb[UB ^ PAR][j][ks]), __builtin_bit_cast(bf16x8, ra[UA][i][ks]),
          acc[2 * UA + i][2 * UB + j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (n < 12) {
        if constexpr (n % 3 == 2) load1(std::integral_constant<int, n / 3>{});
        else rd(std::integral_constant<int, n - n / 3>{});
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    step(std::integral_constant<int, 0>{}); step(std::integral_constant<int, 1>{}); step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 3>{});
    step(std::integral_constant<int, 4>{}); step(std::integral_constant<int, 5>{}); step(std::integral_constant<int, 6>{}); step(std::integral_constant<int, 7>{});
    step(std::integral_constant<int, 8>{}); step(std::integral_constant<int, 9>{}); step(std::integral_constant<int, 10>{}); step(std::integral_constant<int, 11>{});
    step(std::integral_constant<int, 12>{}); step(std::integral_constant<int, 13>{}); step(std::integral_constant<int, 14>{}); step(std::integral_constant<int, 15>{});
    wait_and_barrier<24>();            // six phases' loads may be on their way; the unit read next is older
  };
  auto tile = [&](auto par, int t) {
    const int64_t k2 = k_off(t + 2), k3 = k_off(t + 3);
    phase(par, c0, b_base + k2);
    phase(par, c1, b_base + k2);
    phase(par, c2, a_base + k2);
    phase(par, c3, a_base + k3);
  };
#pragma unroll 1
  for (int t = 0; t < nk; t += 2) {
    tile(c0, t);
    tile(c1, t + 1);
  }
  wait_and_barrier<0>();
#pragma unroll
  for (int i = 0; i < 4; ++i)          // (in accumulation registers until here, whatever the epilogue wants)
    asm volatile("" : "+a"(acc[i][0]), "+a"(acc[i][1]), "+a"(acc[i][2]), "+a"(acc[i][3]));

  if constexpr (SPLIT) {               // partial sums in register order: 1 KB per store
    if (wn == 1 && !second) return;
    float4* dst = static_cast<float4*>(a.part) +
                  (((int64_t)split * a.n_tiles + 2 * b_tile + wn) * (8 * a.m_tiles) + 8 * m_tile + 4 * wm) * 1024 + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          dst[i * 1024 + (4 * j + q) * 64] = make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
    return;
  }
  // epilogue, every wave by itself in 32 KB of the ring's space (nobody reads or fills the ring any more)
  float2* sRho = reinterpret_cast<float2*>(smem + 2 * C::STAGE);
  if (is_rope(EPI) && tid < 64) fill_rho(a, sRho, tid);
  wait_and_barrier<-1>();
  if (wn == 1 && !second) return;
  const OutTile ot = out_tile_of<EPI>(a, block0 + wn);
  if (ot.out) wave_epilogue<4, EPI>(a, ot, acc, sRho, smem + wave * 32768, m0 + wm * 128, lane, rows);
}

typedef WsTile<2, 4, 3> Ws256;         // 256 x 128
typedef WsTile<1, 7, 3> Ws224;         // and so on, as many stages as the LDS holds
typedef WsTile<1, 6, 3> Ws192;
typedef WsTile<1, 5, 4> Ws160;
typedef WsTile<1, 4, 4> Ws128;
typedef WsTile<1, 3, 5> Ws96;
typedef WsTile<1, 2, 6> Ws64;
static_assert(Ws256::BM == rows_of(kWs256) && Ws224::BM == rows_of(kWs224) && Ws192::BM == rows_of(kWs192) && Ws160::BM == rows_of(kWs160) &&
              Ws128::BM == rows_of(kWs128) && Ws96::BM == rows_of(kWs96) && Ws64::BM == rows_of(kWs64) && QuadTile::BN == kQuadCols, "as planned");

// finishes a split launch whose partial sums lie in n_groups groups of 32 rows
template <int EPI>
qcf_status run_split_reduce(const QkvArgs& a, int64_t n_groups, hipStream_t st) {
  const dim3 grid((unsigned)((a.M + 31) / 32), (unsigned)a.n_tiles, 2);
  qkv_split_reduce<EPI><<<grid, dim3(256), 0, st>>>(a, (int)n_groups);
  return check_launch("qkv split reduce");
}

template <typename C, int EPI, bool WIDE>
qcf_status run_ws(QkvArgs a, int splits, hipStream_t st) {
  const int64_t mt = (a.M + C::BM - 1) / C::BM;
  const int nk = a.d_model / kBK;
  a.m_tiles = (int)mt;
  a.splits = splits;
  a.split_len = (nk + splits - 1) / splits;
  const int64_t units = (int64_t)a.n_tiles * splits;
  // Workgroup order.  Few row tiles: all row tiles of a column tile share an XCD, so a weight tile is fetched into
  // one L2 only and the XCD's concurrent workgroups share the row tiles of x.  Many row tiles: an XCD's concurrent
  // workgroups would all belong to one column tile and x would be streamed once per column tile (6 times at 48
  // column tiles); then the row tiles are dealt to the XCDs instead, a row tile of x stays in L2 and the weights
  // are streamed once per row tile (measured at 73 row tiles: 1127 -> 945 us, at 20: 964 -> 912 us).
  a.rows_over_xcds = mt >= kRowsOverXcds;
  const int64_t n_wg = ws_grid(mt, units);
  if (mt > 0x7fffffff || n_wg > 0x7fffffff) return fail(QCF_ERR_UNSUPPORTED, "qkv: grid too large");
  const int64_t side = a.side.rows > 0 ? (a.side.total_rows + a.side.rows - 1) / a.side.rows : 0;
  a.side.first_wg = (int)n_wg;
  static std::atomic<uint64_t> lds_ok;
  QCF_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(&qkv_ws_kernel<C, EPI, WIDE>), C::LDS, lds_ok));
  qkv_ws_kernel<C, EPI, WIDE><<<dim3((unsigned)(n_wg + side)), dim3(C::NTHR), C::LDS, st>>>(a);
  QCF_TRY_LAUNCH("qkv gemm");
  return splits > 1 ? run_split_reduce<EPI>(a, mt * C::NC, st) : QCF_OK;
}

template <int EPI, bool SPLIT>
qcf_status run_quad(QkvArgs a, int splits, hipStream_t st) {
  using C = QuadTile;
  const int64_t mt = (a.M + C::BM - 1) / C::BM;
  const int64_t n_wg = (mt * ((a.n_tiles + 1) / 2) * splits + 255) / 256 * 256;
  if (n_wg > 0x7fffffff) return fail(QCF_ERR_UNSUPPORTED, "qkv: grid too large");
  a.m_tiles = (int)mt;
  const int64_t groups = (mt + 5) / 6;                           // groups of up to six row tiles, of equal size
  a.m_group = (int)((mt + groups - 1) / groups);
  a.splits = splits;
  a.split_len = quad_split_len(a.d_model / kBK, splits);
  static std::atomic<uint64_t> lds_ok;
  QCF_TRY(allow_dynamic_lds(reinterpret_cast<const void*>(&qkv_quad_kernel<EPI, SPLIT>), C::LDS, lds_ok));
  qkv_quad_kernel<EPI, SPLIT><<<dim3((unsigned)n_wg), dim3(C::NTHR), C::LDS, st>>>(a);
  QCF_TRY_LAUNCH("qkv gemm");
  return SPLIT ? run_split_reduce<EPI>(a, mt * 8, st) : QCF_OK;
}

// Product of the generic path.  The small tile reads both operands four times as often, so it takes over only where
// the large one gives fewer workgroups than compute units (M 77, N 512: 16; the small one 160).
bool small_generic(int64_t M, int K, int N) { return (M + 63) / 64 * ((N + 63) / 64) < compute_unit_count() && K % 4 == 0; }
template <typename T, bool ROPE = false>
qcf_status run_gemm_generic(const char* what, const void* x, int64_t x_rows, const int32_t* gather, int64_t M,
                            const void* w, int K, int N, float* y, hipStream_t st, const RopeOut<T>& ro = RopeOut<T>{}) {
  const int64_t mb = (M + 63) / 64;
  const int nb = (N + 63) / 64;
  if (mb > 0x7fffffff || nb > 65535) return fail(QCF_ERR_UNSUPPORTED, "%s: grid too large", what);
  const T* xt = static_cast<const T*>(x);
  const T* wt = static_cast<const T*>(w);
  if (small_generic(M, K, N))
    qkv_gemm_small_generic<T, ROPE><<<dim3((unsigned)((M + 15) / 16), (unsigned)((N + 15) / 16)), dim3(256), 0, st>>>(
        xt, x_rows, gather, M, wt, K, N, y, ro);
  else
    qkv_gemm_generic<T><<<dim3((unsigned)mb, (unsigned)nb), dim3(256), 0, st>>>(xt, x_rows, gather, M, wt, K, N, y);
  return check_launch(what);
}

template <typename T>
qcf_status run_qkv_generic(const qcf_layer_desc& L, const void* x, int64_t x_rows, const int32_t* gather, int64_t M, const void* w,
                           const int32_t* pos, void* q, void* k, void* v, const int32_t* dst_rows, void* k_fused, void* v_fused,
                           int64_t fused_rows, float* y, hipStream_t st) {
  const int heads = L.n_q_heads + 2 * L.n_kv_heads, N = heads * L.head_dim;
  const int64_t rope_blocks = (M * heads * (L.head_dim / 2) + 255) / 256;
  if (rope_blocks > 0x7fffffff) return fail(QCF_ERR_UNSUPPORTED, "qkv: grid too large");
  const RopeOut<T> ro{pos, -2.0 / (double)L.head_dim * std::log2(L.rope_base), L.n_q_heads, L.n_kv_heads, L.head_dim, L.rope_style,
                      static_cast<T*>(q), static_cast<T*>(k), static_cast<T*>(v), dst_rows, static_cast<T*>(k_fused),
                      static_cast<T*>(v_fused), fused_rows};
  if (small_generic(M, L.d_model, N)) return run_gemm_generic<T, true>("qkv", x, x_rows, gather, M, w, L.d_model, N, y, st, ro);
  QCF_TRY(run_gemm_generic<T>("qkv", x, x_rows, gather, M, w, L.d_model, N, y, st));
  qkv_rope_split_generic<T><<<dim3((unsigned)rope_blocks), dim3(256), 0, st>>>(y, M, ro);
  return check_launch("qkv rope");
}

template <int EPI>
qcf_status run_kind(const QkvArgs& a, GemmKind kind, int splits, hipStream_t st) {
  switch (kind) {
    case kQuad: return splits > 1 ? run_quad<EPI, true>(a, splits, st) : run_quad<EPI, false>(a, 1, st);
    case kWs64: return run_ws<Ws64, EPI, false>(a, splits, st);
    case kWs96: return run_ws<Ws96, EPI, false>(a, 1, st);
    case kWs128: return run_ws<Ws128, EPI, false>(a, splits, st);
    case kWs160: return run_ws<Ws160, EPI, false>(a, 1, st);
    case kWs192: return run_ws<Ws192, EPI, false>(a, 1, st);
    case kWs224: return run_ws<Ws224, EPI, false>(a, 1, st);
    default: return run_ws<Ws256, EPI, false>(a, splits, st);
  }
}

template <int EPI>
qcf_status run_gemm(const QkvArgs& a_in, int nb, void* ws, size_t ws_bytes, hipStream_t st) {
  QkvArgs a = a_in;
  const int nk = a.d_model / kBK;
  const bool wide = (uint64_t)a.x_rows * (uint64_t)a.d_model * 2u >= (1ull << 32);
  a.n_tile0 = 0;
  a.n_tiles = nb;
  a.part = ws;
  // (x of 4 GiB and more needs 64-bit addresses per lane: one variant, such calls have plenty of rows)
  if (wide) return run_ws<Ws128, EPI, true>(a, 1, st);
  // (rows that x does not have read its first row: x must not be moved then)
  const ProductPlan p = plan_product(a.M, nb, nk, a.gather || a.x_rows >= a.M, ws_bytes, a.side.rows == 0);
  if (p.blocks == 0) return run_kind<EPI>(a, p.rest.kind, p.rest.splits, st);
  QkvArgs first = a;
  first.M = p.rows;
  first.n_tiles = p.blocks;
  QCF_TRY(run_kind<EPI>(first, p.kind, p.splits, st));
  if (p.rows < a.M) return run_kind<EPI>(rows_from<EPI>(a, p.rows), p.rest.kind, p.rest.splits, st);
  if (p.blocks == nb) return QCF_OK;
  a.n_tile0 = p.blocks;
  a.n_tiles = nb - p.blocks;
  return run_kind<EPI>(a, p.rest.kind, p.rest.splits, st);
}

}  // namespace

size_t qkv_workspace(const qcf_layer_desc& L, int64_t M) {
  // (the MFMA path needs none; what it asks for lets small M split the contraction)
  if (use_mfma(L)) return gemm_part_bytes(M, (L.n_q_heads + 2 * L.n_kv_heads) * L.head_dim / kBN, L.d_model / kBK);
  return align_up((size_t)M * (L.n_q_heads + 2 * L.n_kv_heads) * L.head_dim * sizeof(float), 256);
}

size_t qkv_workspace_needed(const qcf_layer_desc& L, int64_t M) { return use_mfma(L) ? 0 : qkv_workspace(L, M); }

qcf_status launch_qkv(const qcf_layer_desc& L, const void* x, int64_t x_rows, const int32_t* gather,
                      int64_t M, const void* w, const int32_t* pos, void* q, void* k, void* v,
                      const int32_t* dst_rows, void* k_fused, void* v_fused, int64_t fused_rows, void* ws,
                      size_t ws_bytes, hipStream_t st, const SideRerope* side) {
  const int H = L.n_q_heads, Hkv = L.n_kv_heads, D = L.head_dim;
  const int Ntot = (H + 2 * Hkv) * D;
  if (use_mfma(L)) {
    QkvArgs a{};
    if (side) a.side = *side;
    a.x = static_cast<const bf16_t*>(x);
    a.w = static_cast<const bf16_t*>(w);
    a.gather = gather;
    a.pos = pos;
    a.neg2_over_d_log2base = -2.0 / (double)D * std::log2(L.rope_base);
    a.x_rows = x_rows;
    a.M = M;
    a.d_model = L.d_model; a.H = H; a.Hkv = Hkv; a.D = D;
    a.q = static_cast<bf16_t*>(q); a.k = static_cast<bf16_t*>(k); a.v = static_cast<bf16_t*>(v);
    a.dst_rows = dst_rows; a.k_fused = static_cast<bf16_t*>(k_fused); a.v_fused = static_cast<bf16_t*>(v_fused);
    a.fused_rows = fused_rows;
    if (L.rope_style != 0) return run_gemm<kRopeInter>(a, Ntot / kBN, ws, ws_bytes, st);
    if (D == 128) return run_gemm<kRopeHalf128>(a, Ntot / kBN, ws, ws_bytes, st);
    return run_gemm<kRopeHalf64>(a, Ntot / kBN, ws, ws_bytes, st);
  }
  float* y = static_cast<float*>(ws);
  if (L.dtype == QCF_DTYPE_BF16)
    return run_qkv_generic<bf16_t>(L, x, x_rows, gather, M, w, pos, q, k, v, dst_rows, k_fused, v_fused, fused_rows, y, st);
  return run_qkv_generic<float>(L, x, x_rows, gather, M, w, pos, q, k, v, dst_rows, k_fused, v_fused, fused_rows, y, st);
}

qcf_status launch_rerope_qkv(const qcf_layer_desc& L, const qcf_chunk* chunks, int32_t n_chunks, const void* x, int64_t x_rows,
                             const int32_t* gather, int64_t M, const void* w, const int32_t* pos, void* q, void* k, void* v,
                             const int32_t* dst_rows, void* k_fused, void* v_fused, int64_t fused_rows, void* rerope_ws, void* ws,
                             size_t ws_bytes, hipStream_t st) {
  const SideRows rows = side_rows(L, M, n_chunks, fused_rows, ws_bytes);
  if (rows.all < fused_rows) QCF_TRY(launch_rerope(L, chunks, n_chunks, fused_rows, k_fused, v_fused, rerope_ws, st, rows.all));
  const SideRerope side{chunks, rows.all, n_chunks, L.rope_style, 0, (int)rows.each};
  return launch_qkv(L, x, x_rows, gather, M, w, pos, q, k, v, dst_rows, k_fused, v_fused, fused_rows, ws, ws_bytes, st,
                    rows.all > 0 ? &side : nullptr);
}

// ---- plain linear map, RMSNorm, gated SiLU (rest of the layer for the recomputed rows) -----------------

static bool linear_uses_mfma(const qcf_layer_desc& L, int32_t K, int32_t N) {
  return L.dtype == QCF_DTYPE_BF16 && K % kBK == 0 && N % kBN == 0;
}

size_t linear_workspace(const qcf_layer_desc& L, int64_t M, int32_t K, int32_t N) {
  if (linear_uses_mfma(L, K, N)) return gemm_part_bytes(M, N / kBN, K / kBK);       // (optional, see qkv_workspace)
  return align_up((size_t)M * N * sizeof(float), 256);
}

size_t linear_workspace_needed(const qcf_layer_desc& L, int64_t M, int32_t K, int32_t N) {
  return linear_uses_mfma(L, K, N) ? 0 : linear_workspace(L, M, K, N);
}

qcf_status launch_linear(const qcf_layer_desc& L, const void* x, int64_t M, int32_t K, const void* w, int32_t N,
                         const void* residual, void* out, void* ws, size_t ws_bytes, hipStream_t st) {
  if (linear_uses_mfma(L, K, N)) {
    // the projection GEMM with one "query" output of N / 128 heads of 128 columns and no rotation
    QkvArgs a{};
    a.x = static_cast<const bf16_t*>(x);
    a.w = static_cast<const bf16_t*>(w);
    a.x_rows = M;
    a.M = M;
    a.d_model = K; a.H = N / kBN; a.D = kBN;
    a.q = static_cast<bf16_t*>(out);
    a.residual = static_cast<const bf16_t*>(residual);
    return residual ? run_gemm<kAdd>(a, N / kBN, ws, ws_bytes, st) : run_gemm<kPlain>(a, N / kBN, ws, ws_bytes, st);
  }
  float* y = static_cast<float*>(ws);
  const int64_t n = M * N;
  if ((n + 255) / 256 > 0x7fffffff) return fail(QCF_ERR_UNSUPPORTED, "linear: grid too large");
  if (L.dtype == QCF_DTYPE_BF16) {
    QCF_TRY(run_gemm_generic<bf16_t>("linear", x, M, nullptr, M, w, K, N, y, st));
    linear_finish_generic<bf16_t><<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(
        y, static_cast<const bf16_t*>(residual), n, static_cast<bf16_t*>(out));
  } else {
    QCF_TRY(run_gemm_generic<float>("linear", x, M, nullptr, M, w, K, N, y, st));
    linear_finish_generic<float><<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st>>>(
        y, static_cast<const float*>(residual), n, static_cast<float*>(out));
  }
  return check_launch("linear finish");
}

qcf_status launch_rmsnorm(const qcf_layer_desc& L, const void* x, const void* weight, double eps, int64_t M,
                          int32_t cols, void* out, hipStream_t st) {
  if (M > 0x7fffffff) return fail(QCF_ERR_UNSUPPORTED, "rmsnorm: too many rows");
  const dim3 grid((unsigned)M), block(256);
  if (L.dtype == QCF_DTYPE_BF16)
    rmsnorm_kernel<bf16_t><<<grid, block, 0, st>>>(static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(weight),
                                                   (float)eps, cols, static_cast<bf16_t*>(out));
  else
    rmsnorm_kernel<float><<<grid, block, 0, st>>>(static_cast<const float*>(x), static_cast<const float*>(weight),
                                                  (float)eps, cols, static_cast<float*>(out));
  return check_launch("rmsnorm");
}

qcf_status launch_swiglu(const qcf_layer_desc& L, const void* gate_up, int64_t M, int32_t F, void* out,
                         hipStream_t st) {
  const int vec = 16 / elem_size(L.dtype);
  const int64_t blocks = (M * (F / vec) + 255) / 256;
  if (blocks > 0x7fffffff) return fail(QCF_ERR_UNSUPPORTED, "swiglu: too many elements");
  if (L.dtype == QCF_DTYPE_BF16)
    swiglu_kernel<bf16_t><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(static_cast<const bf16_t*>(gate_up), M, F,
                                                                        static_cast<bf16_t*>(out));
  else
    swiglu_kernel<float><<<dim3((unsigned)blocks), dim3(256), 0, st>>>(static_cast<const float*>(gate_up), M, F,
                                                                       static_cast<float*>(out));
  return check_launch("swiglu");
}

// Gate and up columns side by side in the tiles (64 of each per 128-column block): the activation is taken in the
// epilogue, and the product [M, 2F] is neither written nor read again.  Lane offsets into the weights are 32-bit from
// a block's first gate row, which bounds F * K.
// Layer tail with d_model 4096, F 14336: 1229 rows 500 us with a pass of its own for the activation, 480 here; 61 rows
// 121 and 114.
static bool swiglu_in_epilogue(const qcf_layer_desc& L, int32_t K, int32_t F) {
  return linear_uses_mfma(L, K, 2 * F) && F % (kBN / 2) == 0 && ((uint64_t)F + kBN) * (uint64_t)K * 2u < (1ull << 32);
}

static size_t gate_up_bytes(const qcf_layer_desc& L, int64_t M, int32_t F) {
  return align_up((size_t)M * 2 * F * elem_size(L.dtype), 256);
}

size_t linear_swiglu_workspace(const qcf_layer_desc& L, int64_t M, int32_t K, int32_t F) {
  if (swiglu_in_epilogue(L, K, F)) return gemm_part_bytes(M, 2 * F / kBN, K / kBK);       // (optional, see qkv_workspace)
  return gate_up_bytes(L, M, F) + linear_workspace(L, M, K, 2 * F);
}

size_t linear_swiglu_workspace_needed(const qcf_layer_desc& L, int64_t M, int32_t K, int32_t F) {
  return swiglu_in_epilogue(L, K, F) ? 0 : gate_up_bytes(L, M, F) + linear_workspace_needed(L, M, K, 2 * F);
}

qcf_status launch_linear_swiglu(const qcf_layer_desc& L, const void* x, int64_t M, int32_t K, const void* w, int32_t F,
                                void* out, void* ws, size_t ws_bytes, hipStream_t st) {
  if (swiglu_in_epilogue(L, K, F)) {
    QkvArgs a{};
    a.x = static_cast<const bf16_t*>(x);
    a.w = static_cast<const bf16_t*>(w);
    a.x_rows = M;
    a.M = M;
    a.d_model = K;
    a.q = static_cast<bf16_t*>(out);
    a.glu = F;
    return run_gemm<kGlu>(a, 2 * F / kBN, ws, ws_bytes, st);
  }
  const size_t gu = gate_up_bytes(L, M, F);
  QCF_TRY(launch_linear(L, x, M, K, w, 2 * F, nullptr, ws, static_cast<char*>(ws) + gu, ws_bytes - gu, st));
  return launch_swiglu(L, ws, M, F, out, st);
}

}  // namespace qcf
