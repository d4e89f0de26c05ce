/*
 * gemm_workspace.h -- the bf16 matrix product (gemm.h) with caller-owned memory for results of few tiles.
 */
#ifndef GEMM_WORKSPACE_MI355X_H
#define GEMM_WORKSPACE_MI355X_H

#include <stddef.h>

#include "gemm.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * A result of few tiles (a linear layer while decoding, a long reduction) leaves most of the chip idle unless k is cut
 * over workgroups too, whose fp32 partial sums need memory.  gemm_bf16_workspace is gemm_bf16_tile with that memory,
 * owned by the caller: DEVICE memory, 16-byte aligned, contents irrelevant before and after; calls that overlap need one
 * each.  gemm_bf16_workspace_bytes says how much the library's own cut takes (0: none helps; host arithmetic only).
 * splits: workgroups along k of a tile, 0 = the library's choice, at most 64 (a cut finer than k allows is made
 * coarser); splits > 1 needs 4 * M * N * splits bytes.  With a NULL or too small workspace, and for operands the aligned
 * matrix-core kernel does not take (gemm.h), the call is gemm_bf16_tile: the same result up to the order of the fp32
 * sum.  The parts are added in a fixed order: results do not vary from run to run.
 */
size_t gemm_bf16_workspace_bytes(int M, int N, int K);

int gemm_bf16_workspace(const void *a, const void *b, void *c, int M, int N, int K,
                        long long lda, long long ldb, long long ldc, int b_is_nk, int tile, int splits,
                        void *workspace, size_t workspace_bytes, void *stream);

#ifdef __cplusplus
}
#endif
#endif
