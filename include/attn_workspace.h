/*
 * attn_workspace.h -- attention forward (attn.h) with caller-owned memory for calls with few query rows.
 */
#ifndef ATTN_WORKSPACE_MI355X_H
#define ATTN_WORKSPACE_MI355X_H

#include <stddef.h>

#include "attn.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Calls with few query rows (decoding, a few speculated tokens, the tail of a prompt: Sq <= 64 against more than 128
 * keys) have too few (batch, kv head) pairs to fill the chip, and so have longer queries of few heads against long
 * caches (at most 160 blocks of 128 query rows): their keys are cut over workgroups, whose fp32 partial results need
 * memory.  attn_fwd_workspace is attn_fwd_strided with that memory, owned by the caller: DEVICE memory, 16-byte aligned,
 * contents irrelevant before and after; calls that overlap need one each.
 * attn_fwd_workspace_bytes says how much the library's own cut takes (0: none helps; host arithmetic only).
 * splits: workgroups along the keys of a kv head, 0 = the library's choice, at most 256 (a cut finer than the keys
 * allow leaves the surplus parts empty); splits > 1 needs 4 * B * Hq * Sq * splits * (D + 2) bytes.  With a NULL or too
 * small workspace, with splits = 1, and in attn_fwd and attn_fwd_strided, the keys are not cut: the call runs on
 * whichever kernel is the fastest without, to the same result up to the order of fp32 sums.  Other shapes ignore
 * workspace and splits.  ATTN_ERR_UNSUPPORTED: splits out of range; ATTN_ERR_MISALIGNED also covers the workspace.
 */
size_t attn_fwd_workspace_bytes(int B, int Hq, int Hkv, int Sq, int Sk, int D);
int attn_fwd_workspace(const void *q, const void *k, const void *v, void *o, float *lse,
                       int B, int Hq, int Hkv, int Sq, int Sk, int D,
                       const long long *q_strides, const long long *k_strides,
                       const long long *v_strides, const long long *o_strides,
                       int causal, float scale, void *workspace, size_t workspace_bytes, int splits, void *stream);

#ifdef __cplusplus
}
#endif
#endif /* ATTN_WORKSPACE_MI355X_H */
