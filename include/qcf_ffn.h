/*
 * qcf_ffn.h - first half of the gated SiLU feed-forward in one call (conventions of qcf.h).
 */
#ifndef QCF_FFN_H
#define QCF_FFN_H

#include "qcf.h"

#ifdef __cplusplus
extern "C" {
#endif

/* out[m, f] = silu(g) * u with g = x[m, :] . w[f, :] and u = x[m, :] . w[F + f, :], both rounded to the element
 * type first: qcf_linear with N = 2F followed by qcf_swiglu.  x [M, K], w [2F, K] (gate rows, then up rows),
 * out [M, F]; K and F multiples of 8.  One pass on the MFMA path when dtype is bf16, K % 64 == 0, F % 64 == 0
 * and w is below 8 GiB; the workspace is optional there, and the bits of a row depend on it as those of qcf_linear do (only with it
 * on the number of rows).  Otherwise the product [M, 2F] goes through the workspace. */
size_t qcf_linear_swiglu_workspace_bytes(const qcf_layer_desc* desc, int64_t M, int32_t K, int32_t F);
qcf_status qcf_linear_swiglu(const qcf_layer_desc* desc, const void* x, int64_t M, int32_t K, const void* w,
                             int32_t F, void* out, void* workspace, size_t workspace_bytes, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* QCF_FFN_H */
