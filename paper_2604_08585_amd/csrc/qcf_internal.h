// Internal declarations shared by the library's translation units (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <algorithm>
#include <cmath>
#include <atomic>

#include "qcf.h"
#include "qcf_ffn.h"
#include "qcf_layers.h"
#include "qcf_anchors.h"
#include "qcf_fuse.h"

namespace qcf {

// ---- host-side error reporting ------------------------------------------------
qcf_status fail(qcf_status s, const char* fmt, ...);
qcf_status check_hip(hipError_t e, const char* what);
qcf_status check_launch(const char* what);

#define QCF_TRY(expr)                 \
  do {                                \
    qcf_status _s = (expr);           \
    if (_s != QCF_OK) return _s;      \
  } while (0)
#define QCF_TRY_LAUNCH(what) QCF_TRY(::qcf::check_launch(what))

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Raises a kernel's dynamic-LDS limit, once per device and kernel (`done` is a bit mask over device ids kept by
// the caller, one per kernel; a repeated call from another thread is harmless).
qcf_status allow_dynamic_lds(const void* kernel, size_t bytes, std::atomic<uint64_t>& done);
// Compute units of the device that was current at the first call (256 if none could be asked).
int compute_unit_count();
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline int elem_size(int dtype) { return dtype == QCF_DTYPE_BF16 ? 2 : 4; }

// 16-byte and 8-byte register vectors (native vector types, so they live in registers)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x4 mk4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  u32x4 r = {a, b, c, d};
  return r;
}

// ---- storage types --------------------------------------------------------------
typedef uint16_t bf16_t;   // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t v) {
  return __uint_as_float(static_cast<uint32_t>(v) << 16);
}
// round-to-nearest-even; NaN stays NaN
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<bf16_t>((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return static_cast<bf16_t>(u >> 16);
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return static_cast<uint32_t>(f32_to_bf16(lo)) | (static_cast<uint32_t>(f32_to_bf16(hi)) << 16);
}

template <typename T> struct Elem;
template <> struct Elem<float> {
  static constexpr int kVec = 4;   // elements per 16-byte access
  __device__ static __forceinline__ float load(const float* p) { return *p; }
  __device__ static __forceinline__ void store(float* p, float v) { *p = v; }
};
template <> struct Elem<bf16_t> {
  static constexpr int kVec = 8;
  __device__ static __forceinline__ float load(const bf16_t* p) { return bf16_to_f32(*p); }
  __device__ static __forceinline__ void store(bf16_t* p, float v) { *p = f32_to_bf16(v); }
};

// four consecutive elements (the pointer is a multiple of four elements from a 16-byte aligned one)
template <typename T> struct Quad;
template <> struct Quad<float> {
  __device__ static __forceinline__ void load(const float* p, float* f) {
    const float4 r = *reinterpret_cast<const float4*>(p);
    f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w;
  }
};
template <> struct Quad<bf16_t> {
  __device__ static __forceinline__ void load(const bf16_t* p, float* f) {
    const u32x2 r = *reinterpret_cast<const u32x2*>(p);
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
  }
};

// 16-byte vector <-> float unpacking
template <typename T> struct Vec16;
template <> struct Vec16<float> {
  __device__ static __forceinline__ void unpack(const u32x4& r, float* f) {
    f[0] = __uint_as_float(r.x); f[1] = __uint_as_float(r.y);
    f[2] = __uint_as_float(r.z); f[3] = __uint_as_float(r.w);
  }
  __device__ static __forceinline__ u32x4 pack(const float* f) {
    return mk4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]),
                      __float_as_uint(f[3]));
  }
};
template <> struct Vec16<bf16_t> {
  __device__ static __forceinline__ void unpack(const u32x4& r, float* f) {
    f[0] = __uint_as_float(r.x << 16); f[1] = __uint_as_float(r.x & 0xffff0000u);
    f[2] = __uint_as_float(r.y << 16); f[3] = __uint_as_float(r.y & 0xffff0000u);
    f[4] = __uint_as_float(r.z << 16); f[5] = __uint_as_float(r.z & 0xffff0000u);
    f[6] = __uint_as_float(r.w << 16); f[7] = __uint_as_float(r.w & 0xffff0000u);
  }
  __device__ static __forceinline__ u32x4 pack(const float* f) {
    return mk4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]),
                      pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7]));
  }
};

// ---- re-rotation: what its kernels (rerope.hip, and the joined ones of score.hip and qkv.hip) have to do alike, bit for bit
// a rotary pair turned by (cos, sin): the second product of each is rounded, the first one is fused
__device__ __forceinline__ void turn_pair(float a, float b, float2 w, float& oa, float& ob) {
#pragma clang fp contract(off)
  oa = __builtin_fmaf(a, w.x, -(b * w.y));
  ob = __builtin_fmaf(b, w.x, a * w.y);
}
// (cos, sin) of pair i at an angle of `positions` (a whole number) times its frequency, 2^(i * neg2_over_d_log2base)
__device__ __forceinline__ float2 rotary_pair(double positions, double neg2_over_d_log2base, int i) {
  const double theta = exp2(neg2_over_d_log2base * (double)i);
  double sn, cn;
  sincos(positions * theta, &sn, &cn);
  return make_float2((float)cn, (float)sn);
}
__device__ __forceinline__ float2 shift_pair(const qcf_chunk& c, double neg2_over_d_log2base, int i) {
  return rotary_pair((double)(c.dst_pos0 - c.src_pos0), neg2_over_d_log2base, i);
}
// number of the last of n chunks that starts at or before a row (0 if none); dst_row(c): first row of chunk c
template <typename F>
__device__ __forceinline__ int chunk_of(int n, int64_t row, F&& dst_row) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (dst_row(mid) <= row) lo = mid; else hi = mid - 1;
  }
  return lo;
}
__device__ __forceinline__ int chunk_of(const qcf_chunk* table, int n, int64_t row) {
  return chunk_of(n, row, [&](int c) { return table[c].dst_row; });
}

// ---- gfx950 helpers shared by the MFMA kernels ---------------------------------------
typedef float floatx2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

// two floats -> packed bf16 pair, round-to-nearest-even in hardware (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  const floatx2_t f = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

__device__ __forceinline__ uint32_t lds_offset_of(const void* lds) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)(const_cast<void*>(lds));
}

// 16 bytes per lane from global memory straight into LDS: lane L lands at lds + 16*L (lds is
// wave-uniform).  Issued through inline assembly so that the compiler does not count these among the
// loads it waits for before unrelated LDS reads: callers wait for them themselves
// (__builtin_amdgcn_s_waitcnt(0)) before the barrier that publishes the tile.  M0 (the LDS base of
// such a load) is saved and restored around the instruction.
// Form 1: wave-uniform 64-bit base in scalar registers plus a 32-bit byte offset per lane.
__device__ __forceinline__ void load_to_lds(const void* base, uint32_t lane_off, void* lds) {
  const uint32_t lds_addr = __builtin_amdgcn_readfirstlane((int)lds_offset_of(lds));
  const uint64_t b = (uint64_t)(uintptr_t)base;
  // the builtin returns a signed int: widen through uint32_t, or a low half >= 2^31 would smear ones
  // over the high half of the address
  const uint64_t sb = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  uint32_t saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0)
               : "v"(lane_off), "s"(sb), "s"(lds_addr)
               : "memory");
}
// Form 1 with the LDS destination given as a byte address (wave-uniform).
__device__ __forceinline__ void load_to_lds_at(const void* base, uint32_t lane_off, uint32_t lds_addr_in) {
  const uint32_t lds_addr = __builtin_amdgcn_readfirstlane((int)lds_addr_in);
  const uint64_t b = (uint64_t)(uintptr_t)base;
  const uint64_t sb = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  uint32_t saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0)
               : "v"(lane_off), "s"(sb), "s"(lds_addr)
               : "memory");
}
// Form 2: a full 64-bit address per lane; the LDS destination as a pointer or as a byte address.
__device__ __forceinline__ void load_to_lds_addr_at(const void* gptr, uint32_t lds_addr_in) {
  const uint32_t lds_addr = __builtin_amdgcn_readfirstlane((int)lds_addr_in);
  uint32_t saved_m0;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n\ts_mov_b32 m0, %0"
               : "=&s"(saved_m0)
               : "v"(gptr), "s"(lds_addr)
               : "memory");
}

__device__ __forceinline__ void load_to_lds_addr(const void* gptr, void* lds) { load_to_lds_addr_at(gptr, lds_offset_of(lds)); }

// Form 1 without the compiler-level memory fence (ordinary LDS accesses may be scheduled across it: for loops that
// interleave these loads with fragment reads of another stage and order everything with their own waits and
// barriers), with the LDS destination as wave-uniform base + constant and M0 left as it is.
// (M0 is reserved: the compiler sets it right before each use of its own, so it is not restored here.)
template <int OFF>
__device__ __forceinline__ void load_to_lds_const(const void* base, uint32_t lane_off, uint32_t lds_base) {
  const uint64_t b = (uint64_t)(uintptr_t)base;
  const uint64_t sb = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32) |
                      (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b);
  asm volatile("s_add_u32 m0, %2, %3\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :: "v"(lane_off), "s"(sb), "s"(lds_base), "n"(OFF) : "scc");
}

// sums over the 16 lanes of each row and the 32 of each half of a wave, in a fixed order; every lane gets the total
__device__ __forceinline__ float row_sum(float x) {
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x128, 0xf, 0xf, false));   // row_ror:8
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x124, 0xf, 0xf, false));   // row_ror:4
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x122, 0xf, 0xf, false));   // row_ror:2
  x += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x121, 0xf, 0xf, false));   // row_ror:1
  return x;
}
__device__ __forceinline__ float half_wave_sum(float x) {
  x = row_sum(x);
  typedef unsigned u2v __attribute__((ext_vector_type(2)));
  const u2v r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r.x) + __uint_as_float(r.y);     // rows (0, 1) and (2, 3) of 16 lanes each
}

// sum and maximum over the lanes of a wave; every lane gets it
__device__ __forceinline__ float wave_sum(float x) {
  x = half_wave_sum(x);
  typedef unsigned u2v __attribute__((ext_vector_type(2)));
  const u2v r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r.x) + __uint_as_float(r.y);
}
__device__ __forceinline__ float wave_max(float x) {
  typedef unsigned u2v __attribute__((ext_vector_type(2)));
  x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x128, 0xf, 0xf, false)));
  x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x124, 0xf, 0xf, false)));
  x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x122, 0xf, 0xf, false)));
  x = fmaxf(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x121, 0xf, 0xf, false)));
  u2v r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r.x), __uint_as_float(r.y));
}

// ---- launchers (one per translation unit) --------------------------------------
// Each returns QCF_OK or an error after enqueueing on `st`; arguments were validated
// by the entry points in api.hip.

size_t rerope_workspace(const qcf_layer_desc& L, int32_t n_chunks, int64_t total_rows);
qcf_status launch_rerope(const qcf_layer_desc& L, const qcf_chunk* chunks, int32_t n_chunks,
                         int64_t total_rows, void* kf, void* vf, void* ws, hipStream_t st, int64_t row0 = 0);      // rows from row0 on

// host-side validation shared by the two scoring entry points; *empty = nothing to do
qcf_status check_score_args(const qcf_layer_desc* desc, int32_t B, const void* q_probe,
                            const int64_t* probe_off_dev, int64_t total_probe, const void* k_fused,
                            const int64_t* ctx_off_dev, int64_t total_ctx, const int32_t* probe_limit_dev,
                            float* score, bool* empty);
// The last sums of a scoring that are left to the selection of the same request (launch_score fills it in instead of adding them).
struct ScoreSums {
  const float* sums;             // [n][total_ctx]: of the KV heads, or of every probe row and head (rows)
  const int64_t* probe_off;
  int64_t total_probe;
  int H, Hkv;
  bool rows;
};
qcf_status launch_score(const qcf_layer_desc& L, int32_t B, const void* q, const int64_t* probe_off,
                        int64_t total_probe, const void* k, const int64_t* ctx_off, int64_t total_ctx,
                        const int32_t* probe_limit, float* score, float alpha, float beta, void* ws, hipStream_t st,
                        ScoreSums* left = nullptr);

// re-rotation and scoring of one request: in one launch where scoring::takes_rerope, the re-rotation inside the first of the two
// passes (two launches, three where the last sums are not left to the selection) where scoring::pass1_takes_rerope
qcf_status launch_rerope_score(const qcf_layer_desc& L, const qcf_chunk* chunks, int32_t n_chunks, const void* q,
                               const int64_t* probe_off, int64_t total_probe, void* k, void* v, const int64_t* ctx_off,
                               int64_t total_ctx, float* score, void* ws, hipStream_t st, ScoreSums* left);

qcf_status launch_score_layers(const qcf_layer_desc& L, int32_t n_layers, int32_t B, const void* const* q,
                               const int64_t* probe_off, int64_t total_probe, const void* const* k, const int64_t* ctx_off,
                               int64_t total_ctx, const int32_t* probe_limit, const float* weights, float* score, void* ws,
                               hipStream_t st);

size_t select_workspace(int32_t B, int64_t total_ctx);
qcf_status launch_select(int32_t B, const float* score, const int64_t* ctx_off, int64_t total_ctx,
                         const int64_t* sel_off, int64_t total_sel, const int32_t* ctx_pos0,
                         int32_t* sel_idx, int32_t* sel_row, int32_t* sel_pos, void* ws,
                         hipStream_t st);

// the last sums of a scoring (launch_score with `left`), its scores and the selection over them; the offsets are device arrays
qcf_status launch_select_sums(const ScoreSums& sums, float* score, const int64_t* ctx_off, int64_t total_ctx, const int64_t* sel_off,
                              int64_t total_sel, int32_t* sel_idx, int32_t* sel_row, int32_t* sel_pos, hipStream_t st);
// Top-N of every chunk and the gather of its key and value rows; the offsets are host arrays
qcf_status launch_select_gather(const qcf_layer_desc& L, const float* score, int32_t n_chunks, const int64_t* ctx_off,
                                const int64_t* sel_off, const void* k, const void* v, int32_t* rows, void* k_out, void* v_out,
                                hipStream_t st);

size_t qkv_workspace(const qcf_layer_desc& L, int64_t M);
// dst_rows / k_fused / v_fused (all or none): the K/V rows are also written to rows dst_rows[m] of the fused cache
qcf_status launch_qkv(const qcf_layer_desc& L, const void* x, int64_t x_rows, const int32_t* gather,
                      int64_t M, const void* w, const int32_t* pos, void* q, void* k, void* v,
                      const int32_t* dst_rows, void* k_fused, void* v_fused, int64_t fused_rows,
                      void* ws, size_t ws_bytes, hipStream_t st, const struct SideRerope* side = nullptr);
// qcf_rerope (keys and values; rerope_ws) and the same, the one beside the other where the launch has compute units to spare
qcf_status launch_rerope_qkv(const qcf_layer_desc& L, const qcf_chunk* chunks, int32_t n_chunks, const void* x, int64_t x_rows,
                             const int32_t* gather, int64_t M, const void* w, const int32_t* pos, void* q, void* k, void* v,
                             const int32_t* dst_rows, void* k_fused, void* v_fused, int64_t fused_rows, void* rerope_ws, void* ws,
                             size_t ws_bytes, hipStream_t st);

qcf_status launch_scatter(const qcf_layer_desc& L, const void* k_new, const void* v_new,
                          const int32_t* rows, int64_t M, void* kf, void* vf, int64_t total_rows,
                          hipStream_t st);

qcf_status launch_gather(const qcf_layer_desc& L, const void* k_src, const void* v_src, const int32_t* rows,
                         int64_t M, int64_t src_rows, void* k_out, void* v_out, hipStream_t st);
qcf_status launch_key_norm(const qcf_layer_desc& L, const void* k, int64_t rows, float* norm, hipStream_t st);

size_t attn_workspace(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx);
qcf_status launch_attn(const qcf_layer_desc& L, int32_t B, const void* q, const int32_t* sel_pos,
                       const int64_t* sel_off, int64_t total_sel, const void* k, const void* v,
                       const int64_t* ctx_off, int64_t total_ctx, const int32_t* ctx_pos0, void* o,
                       float* lse, void* ws, size_t ws_bytes, hipStream_t st);

size_t linear_workspace(const qcf_layer_desc& L, int64_t M, int32_t K, int32_t N);
qcf_status launch_linear(const qcf_layer_desc& L, const void* x, int64_t M, int32_t K, const void* w, int32_t N,
                         const void* residual, void* out, void* ws, size_t ws_bytes, hipStream_t st);
size_t linear_swiglu_workspace(const qcf_layer_desc& L, int64_t M, int32_t K, int32_t F);
qcf_status launch_linear_swiglu(const qcf_layer_desc& L, const void* x, int64_t M, int32_t K, const void* w, int32_t F,
                                void* out, void* ws, size_t ws_bytes, hipStream_t st);
// bytes a call cannot do without (the rest of the workspace only makes it faster)
size_t qkv_workspace_needed(const qcf_layer_desc& L, int64_t M);
size_t attn_workspace_needed(const qcf_layer_desc& L, int32_t B, int64_t total_sel, int64_t total_ctx);
size_t linear_workspace_needed(const qcf_layer_desc& L, int64_t M, int32_t K, int32_t N);
size_t linear_swiglu_workspace_needed(const qcf_layer_desc& L, int64_t M, int32_t K, int32_t F);
qcf_status launch_rmsnorm(const qcf_layer_desc& L, const void* x, const void* weight, double eps, int64_t M,
                          int32_t cols, void* out, hipStream_t st);
qcf_status launch_swiglu(const qcf_layer_desc& L, const void* gate_up, int64_t M, int32_t F, void* out,
                         hipStream_t st);

}  // namespace qcf
