// Internal interface between the C-ABI translation unit (argument checks, no device
// code) and the GEMM kernel translation unit.
#pragma once
#include <hip/hip_runtime.h>

struct GemmParams {
    const __bf16* a;   // [M, K], row pitch lda
    const __bf16* b;   // [K, N] (row pitch ldb) or, if b_is_nk, [N, K]
    __bf16* c;         // [M, N], row pitch ldc
    int M, N, K;
    long long lda, ldb, ldc;   // elements
    int tiles_m, tiles_n;      // set by the launcher for the kernel it picks
    int splits, split_stages;  // workgroups along k of a tile, and the stages each of them takes (set by the launcher)
    float* part;               // splits > 1: [splits, M, N] fp32 parts
};

// The workgroup tile gemm_launch takes for an M x N result when the caller leaves the choice open
// (64, 128, 1284 or 256: see gemm_bf16_tile in include/gemm.h).  Host arithmetic only.
int gemm_auto_tile(int M, int N);

// Workgroup tile and workgroups along k for a call that has memory for parts; tile and splits 0: by size.
constexpr int kMaxGemmSplits = 64;
struct GemmPlan { int tile, splits; };
GemmPlan gemm_plan(int M, int N, int K, int tile, int splits);
inline size_t gemm_plan_bytes(int M, int N, GemmPlan plan) { return plan.splits <= 1 ? 0 : (size_t)M * N * plan.splits * sizeof(float); }

// Enqueue the product on `stream`; `tiled` says whether the operands satisfy the
// alignment rules of the matrix-core kernel; `tile` is 0 (gemm_auto_tile) or one of the values
// gemm_bf16_tile accepts.  Returns 0, or -1 if the launch was refused.
int gemm_launch(GemmParams p, int b_is_nk, bool tiled, int tile, hipStream_t stream);

// Operands that fail those alignment rules: whether the register-fed matrix-core kernel takes these sizes, and its
// launch; `tile` as `asked` of unaligned_tile (gemm_layout.h).
bool gemm_unaligned_sizes(int N, int K, int b_is_nk);
void gemm_unaligned_launch(const GemmParams& p, int b_is_nk, int tile, hipStream_t stream);
