// Internal interface between the C-ABI translation unit (argument checks, no device
// code) and the kernel translation unit.
#pragma once
#include <hip/hip_runtime.h>

struct AttnParams {
    const __bf16* q;
    const __bf16* k;
    const __bf16* v;
    __bf16* o;
    float* lse;        // may be null
    int B, Hq, Hkv, Sq, Sk;
    // element strides: batch, head, sequence row (the D elements of a row are contiguous)
    long long q_sb, q_sh, q_ss, k_sb, k_sh, k_ss, v_sb, v_sh, v_ss, o_sb, o_sh, o_ss;
    int nQt;           // query tiles per head (set by the launcher for the kernel it picks)
    int nblocks;       // B * (Hq / hpw) * nQt  (set by the launcher)
    int hpw, hpw_log2; // query heads of one kv head that a workgroup covers side by side: 1, 2, 4 or 8 (set by the launcher)
    float scale;       // multiplier on q.k before the softmax
    float scale_log2;  // scale * log2(e): scores are exponentiated with exp2
};

// Enqueue the forward kernel for head dimension D (64 or 128) on `stream`.  wg_rows: query rows per workgroup
// of the tiled kernel, 256 or 128, or 0 for the launcher's own choice.
// Returns 0, -1 if the runtime refused the launch, -2 if the grid would not fit 31 bits.
int attn_launch(AttnParams p, int D, int causal, int wg_rows, hipStream_t stream);

// Keys of one kv head cut over workgroups (attn_split_kernel.hip): the path of calls with few query rows or few heads.
constexpr int kMaxSplits = 256;
struct AttnSplit {
    int rb;            // 32-row blocks of packed query rows per workgroup: 1, 2 or 4
    int waves;         // wavefronts per workgroup: 4, or 2 (rb = 1)
    int row_wgs;       // workgroups along the packed query rows of a kv head
    int splits;        // workgroups along its keys
    double cost;       // estimated time, microseconds
    float* part;       // [B*Hq*Sq, splits, D] unnormalised O of every split, relative to its own maximum
    float* ml;         // [B*Hq*Sq, splits, 2] that maximum (raw score units) and the row sum
};
// Whether the call's shape is one for that path: with or without memory for parts (few query rows), or with it (a grid of
// tiles that would leave most of the chip idle); and whether its strides are.
bool attn_split_sizes(int Sq, int Sk);
bool attn_split_pays(int B, int Hq, int Hkv, int Sq, int Sk, int D);
bool attn_split_fits(const AttnParams& p);
// Up to 64 query positions: whether that cut is faster than the 128-row kernel.
bool attn_split_wins(const AttnSplit& sp, int B, int Hq, int Sk, int D);
// Its cut; splits 0: by size.  Host arithmetic only.
AttnSplit attn_split_plan(int B, int Hq, int Hkv, int Sq, int Sk, int D, int splits);
// Bytes of workspace that cut needs: none for one split.
size_t attn_split_bytes(int B, int Hq, int Sq, int D, int splits);
int attn_split_launch(AttnParams p, int D, int causal, AttnSplit sp, void* workspace, hipStream_t stream);

// Enqueue the pure-MFMA calibration kernel (blocks x 8 wavefronts x iters x 4 MFMAs); returns
// the FLOPs it performs, or -1 if the launch was refused.  sink: >= 4 bytes of device memory.
double attn_launch_mfma_calibration(float* sink, int blocks, int iters, int data, hipStream_t stream);
