/*
 * qcf_anchors.h - summary anchors of stored chunks in one call (conventions of qcf.h).
 */
#ifndef QCF_ANCHORS_H
#define QCF_ANCHORS_H

#include "qcf.h"

#ifdef __cplusplus
extern "C" {
#endif

/* For chunks stored back to back in k and v ([total rows, H_kv, d]): the rows of each chunk with the largest key norm,
 * ascending, and their keys and values: what qcf_key_norm, qcf_select (sel_row) and qcf_gather give one after the other.
 * Chunk c holds rows ctx_off[c] .. ctx_off[c+1] - 1 and gives outputs sel_off[c] .. sel_off[c+1] - 1.  Both are HOST
 * arrays of n_chunks + 1 entries, read before the call returns; their last entries are the totals. */
size_t qcf_extract_anchors_workspace_bytes(const qcf_layer_desc* desc, int32_t n_chunks, int64_t total_rows);
qcf_status qcf_extract_anchors(const qcf_layer_desc* desc, const void* k, const void* v, int32_t n_chunks,
                               const int64_t* ctx_off, const int64_t* sel_off, int32_t* rows, void* k_out, void* v_out,
                               void* workspace, size_t workspace_bytes, void* stream);

#ifdef __cplusplus
}
#endif
#endif /* QCF_ANCHORS_H */
