/*
 * qcf_layers.h - scores of several layers in one call (conventions of qcf.h).
 */
#ifndef QCF_LAYERS_H
#define QCF_LAYERS_H

#include "qcf.h"

#ifdef __cplusplus
extern "C" {
#endif

/* score[j] = sum over layers l, in order, of weights[l] * (mean attention of layer l's probe rows on token j): what
 * qcf_score_accumulate gives called once per layer, the first time with beta = 0, then with beta = 1.  q_probe, k_fused
 * and weights are HOST arrays of n_layers entries (device pointers, floats), read before the call returns; the offsets,
 * totals and probe_limit are those of every layer.  n_layers >= 1.  bf16 with head_dim 128: several layers share their
 * launches, and everything stays in the workspace.  Deterministic. */
size_t qcf_score_layers_workspace_bytes(const qcf_layer_desc* desc, int32_t n_layers, int32_t B, int64_t total_probe,
                                        int64_t total_ctx);
qcf_status qcf_score_layers(const qcf_layer_desc* desc, int32_t n_layers, int32_t B, const void* const* q_probe,
                            const int64_t* probe_off_dev, int64_t total_probe, const void* const* k_fused,
                            const int64_t* ctx_off_dev, int64_t total_ctx, const int32_t* probe_limit_dev,
                            const float* weights, float* score, void* workspace, size_t workspace_bytes, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* QCF_LAYERS_H */
