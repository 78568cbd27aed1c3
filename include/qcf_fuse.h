/*
 * qcf_fuse.h - one layer of the path in one call (conventions of qcf.h).
 */
#ifndef QCF_FUSE_H
#define QCF_FUSE_H

#include "qcf.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Buffers of one layer (host struct, read before the call returns).  Sizes and meanings are those of the calls of qcf.h; x holds
 * the hidden states of all total_ctx context rows, positions are rows of the request (no ctx_pos0), and the selected rows are
 * gathered from, and written back to, rows sel_row.  A workspace is the one of the call it is named for. */
typedef struct qcf_layer_buffers {
  int32_t B, n_chunks;
  int64_t total_ctx, total_probe, total_sel;
  const qcf_chunk* chunks_dev;
  const int64_t* ctx_off_dev;
  const int64_t* probe_off_dev;       /* critical layer only, with q_probe, score and sel_idx */
  const int64_t* sel_off_dev;
  const void* q_probe;
  const void* x;
  const void* w_qkv;
  void* k_fused;
  void* v_fused;
  float* score;
  int32_t* sel_idx;
  int32_t* sel_row;                   /* outputs at the critical layer, inputs at the others; so is sel_pos */
  int32_t* sel_pos;
  void* q_sel;
  void* k_sel;
  void* v_sel;
  void* o_sel;
  float* lse;                         /* may be NULL */
  void* rerope_ws;
  void* score_ws;
  void* select_ws;
  void* qkv_ws;
  void* attn_ws;
  size_t rerope_ws_bytes, score_ws_bytes, select_ws_bytes, qkv_ws_bytes, attn_ws_bytes;
} qcf_layer_buffers;

/* qcf_rerope, at the critical layer qcf_score and qcf_select, qcf_recompute_qkv_scatter and qcf_recompute_attn, one after the
 * other: same results, arguments checked call by call.  A call that fails ends the layer; what is in front of it has been
 * enqueued.  Launches may be joined.  At the critical layer: where qcf_score is the one kernel whose workgroups wait for each
 * other, so is its part here, and the keys and values of one request are re-rotated by that kernel, or with heads of 64 by the
 * first pass of two (up to 128 chunks, not of a few tokens each); the last sums of the scores may be the selection's.  At the other
 * layers: the cache rows, or a part of them, are re-rotated by workgroups behind those of the projection, on the compute units that
 * it leaves idle (bf16, up to 256 chunks); rows that the projection writes are left to it. */
qcf_status qcf_fuse_layer(const qcf_layer_desc* desc, const qcf_layer_buffers* layer, int32_t critical, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* QCF_FUSE_H */
