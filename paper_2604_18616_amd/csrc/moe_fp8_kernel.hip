// Fused mixture-of-experts feed-forward in block-quantized FP8 for gfx950 (MI355X): the
// paper's fused-MoE workload (Evaluation, "Kernel Performance", "Fused MoE" paragraph: tokens and experts are
// partitioned, tokens reach their experts through sorted maps, blockwise quantization is
// preserved, the up-projection intermediates are quantized to FP8 so that both projections run
// on the FP8 matrix cores).
//
// Five stages in four kernels on one stream, all state in the caller's workspace:
//   moe_prepare   workgroup 0: counting sort of the local (token, slot) pairs by expert (sorted
//                 rows, the inverse map, one record per row tile); the other workgroups: activation
//                 quantization, eight groups of 128 features per 32 lanes;
//   moe_gemm<UP>  per (row tile, 128 intermediate columns): gate and up products on
//                 v_mfma_f32_16x16x128_f8f6f4, block scales applied per 128-deep stage,
//                 SiLU gate, requantization of the 128-column group, FP8 store;
//   moe_gemm<DN>  per (row tile, 256 output columns, or 128 if that is what it takes to give every CU a
//                 workgroup): down product; the row of a token with a single local slot
//                 goes straight to y (weight * row, rounded once), the others as fp32 rows to the workspace;
//   moe_combine   y[t] = sum over local slots of weight * row, rounded once to bf16, for the tokens with
//                 two or more local slots; zeros for those with none.
// With 16 to 256 rows per expert the products are bound by streaming the expert weights from
// HBM (each byte is used for 2 x rows FLOPs), so the grouped product keeps three 40-52 KB stages
// (two of 56-64 KB for tiles of more than 160 rows) of direct-to-LDS copies per workgroup, all but one of them in flight.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_layout.h"
#include <mutex>

#include "moe_launch.h"
#include "gfx950_prims.h"

namespace {

using namespace gfx950;

using namespace gemm_layout;   // kt_*: the 128-byte-row swizzled tile of the bf16 GEMM, here 128 e4m3 per row

// quant128 on four values of a 32-lane group: returns the four e4m3 codes packed little-endian.
// scale = amax * (1/448) (1 if amax = 0), code = e4m3(clamp(v * (1/scale))): fp32 throughout, a true
// division, v_cvt_pk_fp8_f32 rounds to nearest even (checked against the format on the device).
__device__ __forceinline__ float quant_scale(float amax) { return amax == 0.0f ? 1.0f : amax * (1.0f / 448.0f); }
__device__ __forceinline__ unsigned quant_pack4(float v0, float v1, float v2, float v3, float inv) {
    const float c0 = fminf(fmaxf(v0 * inv, -448.0f), 448.0f), c1 = fminf(fmaxf(v1 * inv, -448.0f), 448.0f);
    const float c2 = fminf(fmaxf(v2 * inv, -448.0f), 448.0f), c3 = fminf(fmaxf(v3 * inv, -448.0f), 448.0f);
    int p = __builtin_amdgcn_cvt_pk_fp8_f32(c0, c1, 0, false);
    p = __builtin_amdgcn_cvt_pk_fp8_f32(c2, c3, p, true);
    return (unsigned)p;
}

// ------------------------------------------------------------------------------------
// Routing: one workgroup of 16 wavefronts.  Thousands of slots land on a few dozen counters, so each
// wavefront counts into a histogram of its own (LDS atomics without a return value); the per-expert
// totals and the wavefronts' shares are turned into start rows by a block-wide scan; the scatter
// pass takes its row from the wavefront's own counter again, so only lanes of one wavefront ever
// contend.  Rows within an expert come out in no particular order: every row is computed on its
// own and found again through `pos`.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void route_block(const MoeParams& p) {
    __shared__ int wcnt[16 * 256];          // [wavefront][expert]: counts, then running row cursors
    __shared__ int rows_scan[256], tiles_scan[256], cnt[256];
    const int tid = threadIdx.x, wave = tid >> 6, E = p.E, n = p.T * p.KTOP;
    for (int i = tid; i < 16 * 256; i += 1024) wcnt[i] = 0;
    __syncthreads();
    // (both passes take kRU slots per thread and iteration with the loads issued together: this workgroup is
    // alone with the latency of its loads, and under the quantization blocks' traffic that latency is long)
    constexpr int kRU = 4;
    for (int i0 = tid; i0 < n; i0 += 1024 * kRU) {
        int e[kRU];
#pragma unroll
        for (int j = 0; j < kRU; ++j) { const int i = i0 + 1024 * j; e[j] = i < n ? p.ids[i] : -1; }
#pragma unroll
        for (int j = 0; j < kRU; ++j) if (e[j] >= 0 && e[j] < E) atomicAdd(&wcnt[wave * 256 + e[j]], 1);
    }
    __syncthreads();
    if (tid < 256) {                         // expert tid: total, and each wavefront's offset inside the expert
        int run = 0;
        if (tid < E)
            for (int w = 0; w < 16; ++w) { const int c = wcnt[w * 256 + tid]; wcnt[w * 256 + tid] = run; run += c; }
        cnt[tid] = run;
        rows_scan[tid] = run;
        tiles_scan[tid] = p.bm ? moe_tiles(run, p.bm) : moe_tiles(run, 128) << 16 | moe_tiles(run, 0);      // (both cuts: at most 8448 tiles)
    }
    __syncthreads();
    for (int d = 1; d < 256; d <<= 1) {      // inclusive scans over the experts
        int r = 0, t = 0;
        if (tid < 256 && tid >= d) { r = rows_scan[tid - d]; t = tiles_scan[tid - d]; }
        __syncthreads();
        if (tid < 256) { rows_scan[tid] += r; tiles_scan[tid] += t; }
        __syncthreads();
    }
    if (tid < E) {
        const int all = tiles_scan[255];
        const int bm = p.bm || rows_scan[255] == 0 ? p.bm : moe_choose(rows_scan[255], all >> 16, all & 0xffff, p.H, p.I);   // uniform
        const int nt = moe_tiles(cnt[tid], bm), upto = p.bm ? tiles_scan[tid] : bm ? tiles_scan[tid] >> 16 : tiles_scan[tid] & 0xffff;
        const int start = rows_scan[tid] - cnt[tid], tstart = upto - nt;
        p.offsets[tid] = start;
        for (int w = 0; w < 16; ++w) wcnt[w * 256 + tid] += start;
        for (int m = 0; m < nt; ++m) {
            p.tile_rec[tstart + m] = MoeTileRec{tid, start, cnt[tid], tstart};
        }
        if (tid == E - 1) { p.offsets[E] = rows_scan[tid]; p.ntiles[0] = upto; p.ntiles[1] = bm; }
    }
    __syncthreads();
    for (int i0 = tid; i0 < n; i0 += 1024 * kRU) {
        int e[kRU];
#pragma unroll
        for (int j = 0; j < kRU; ++j) { const int i = i0 + 1024 * j; e[j] = i < n ? p.ids[i] : -1; }
#pragma unroll
        for (int j = 0; j < kRU; ++j) {
            const int i = i0 + 1024 * j;
            if (i >= n) break;
            int r = -1;
            if (e[j] >= 0 && e[j] < E) {
                r = atomicAdd(&wcnt[wave * 256 + e[j]], 1);
                p.sorted_tok[r] = i / p.KTOP;
            }
            p.pos[i] = r;
        }
    }
}

// ------------------------------------------------------------------------------------
// Activation quantization: 32 lanes per group of 128 features, 4 features per lane.
// ------------------------------------------------------------------------------------
constexpr int kMoeQuantGroups = 8;           // groups of 128 features one 32-lane unit quantizes, all loaded up front (4: 15 % slower)
__device__ __forceinline__ void quant_x_block(const MoeParams& p, unsigned block) {
    // 32 lanes take kQG consecutive groups of one token (all loads issued before the first use)
    constexpr int kQG = kMoeQuantGroups;
    const int gpt = p.H / 128;                                    // groups per token
    const int cpt = (gpt + kQG - 1) / kQG;                        // 32-lane work items per token
    const long long item = (long long)block * 32 + (threadIdx.x >> 5);
    if (item >= (long long)p.T * cpt) return;
    const int t = (int)(item / cpt), g0 = (int)(item - (long long)t * cpt) * kQG;
    {   // tokens without a local slot are never read by the products: skip them
        const int k = threadIdx.x & 31;                           // (at most 16 slots: one load of a lane each)
        const int e = k < p.KTOP ? p.ids[t * p.KTOP + k] : -1;
        const unsigned long long local = __builtin_amdgcn_ballot_w64(e >= 0 && e < p.E);
        if ((unsigned)(threadIdx.x & 32 ? local >> 32 : local) == 0) return;
    }
    const int l = threadIdx.x & 31;
    u32x2 raw[kQG];
#pragma unroll
    for (int q = 0; q < kQG; ++q) raw[q] = *(const u32x2*)(p.x + ((size_t)t * gpt + min(g0 + q, gpt - 1)) * 128 + l * 4);
#pragma unroll
    for (int q = 0; q < kQG; ++q) {
        if (g0 + q >= gpt) break;
        const size_t g = (size_t)t * gpt + g0 + q;
        const float v0 = __uint_as_float(raw[q][0] << 16), v1 = __uint_as_float(raw[q][0] & 0xffff0000u);
        const float v2 = __uint_as_float(raw[q][1] << 16), v3 = __uint_as_float(raw[q][1] & 0xffff0000u);
        float amax = fmaxf(fmaxf(fabsf(v0), fabsf(v1)), fmaxf(fabsf(v2), fabsf(v3)));
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 32));
        const float scale = quant_scale(amax);
        const float inv = 1.0f / scale;
        *(unsigned*)(p.xq + g * 128 + l * 4) = quant_pack4(v0, v1, v2, v3, inv);
        if (l == 0) p.xs[g] = scale;
    }
}

// Stages 0 and 1 do not depend on each other: one launch, workgroup 0 routes while the others quantize.
// `stages` bit 0: routing, bit 1: quantization.
__global__ __launch_bounds__(1024) void moe_prepare(MoeParams p, int stages) {
    if (blockIdx.x == 0) {
        if (stages & 1) route_block(p);
    } else if (stages & 2) {
        quant_x_block(p, blockIdx.x - 1);
    }
}

// ------------------------------------------------------------------------------------
// Grouped block-scaled FP8 product.  Workgroup = 8 wavefronts = 4 (n) x 2 (m) for the MFMAs: 256 weight rows x
// BM routed rows.  An expert's rows are cut into one tile of up to 160, or evenly into the fewest of up to 256 rows
// (moe_tiles), or into tiles of 128 where those fill the chip better (moe_choose, once per call; a caller may ask for 128
// or 64); each workgroup picks the code for BM = 64, 128, 160, 192, 224 or 256 from the rows its tile really has.  Up to 160
// rows the weights come from HBM for that one tile and three LDS stages cover the latency.  From there on two stages fit.
// Wavefront (wn, wm): weight rows 64 wn .. +63 as four 16-row MFMA operands, routed rows (BM/2) wm .. in the lanes, BM/32
// blocks of 16 (transposed product, as in the bf16 GEMM), on v_mfma_f32_16x16x128_f8f6f4: one instruction takes a whole
// stage of k, so a product is scaled and added up as four registers, not sixteen, and can wait for its turn.
//   UP:  the 256 weight rows of column tile nt are, per wavefront, 32 gate rows j and the 32 up
//        rows I + j of the same j: both accumulators of a lane meet the same (row, j).
//   DN:  256 consecutive rows of w2.
// One stage = 128 bytes of k for all rows (BM x 128 routed + 32 KB weights); per stage acc += product * (row scale x weight
// block scale).
// What bounds it: the copies, from HBM while an expert has one row tile, then from L2; with more rows the products, whose LDS
// reads (192 KB per stage of 256 rows) take as long as the matrix pipes do.  Measured, gate/up / down, us, before and after
// row scales by fours instead of a copy per row and stage, weights copied a stage earlier, one product per stage:
// 16384 tokens of (7168 x 2048, 32 experts) 447 / 238 -> 361 / 209; 8192 tokens 205 / 148 -> 183 / 138; 4096 tokens of
// (4096 x 14336, 8 experts) 1100 / 672 -> 1000 / 555; (2048 x 768, 128 experts) 172 / 160 -> 160 / 149.  With the copies alone
// the first takes 376 (before), with the products alone 278.
// ------------------------------------------------------------------------------------
constexpr int kMoeBN = 256;
constexpr int kMoeLdsBytes = 3 * (160 * 128 + kMoeBN * 128);   // the largest stage set: three stages of BM = 160
constexpr int kMoeFewLdsBytes = 3 * 32 * 128 + 2 * kMoeBN * 128;   // of a workgroup with BM = 32
constexpr int kMoeScaleBytes = 2 * 2 * 160 * 4;               // scale products of two stages for up to 160 rows; those of more lie behind two stages of tiles
constexpr int kMoeMaxKB = 128;                      // 128-blocks along k: H, I <= 16384

typedef __attribute__((address_space(3))) char* LdsChar;      // LDS pointers stay typed as such: a generic pointer would
typedef __attribute__((address_space(3))) float* LdsFloat;    // turn the scale reads into flat loads, which count as vector memory
template <bool UP, int BM, int BN>
__device__ __forceinline__ void moe_gemm_tile(const MoeParams& p, int e, int row0, int rows, int nt, bool few, LdsChar smem, LdsFloat scales, LdsFloat sb_tab) {
    static_assert(BN == 256 || (BN == 128 && !UP), "the gate/up product pairs gate and up rows per wavefront");
    // LDS stages of the weights and of the routed rows: what 160 KB hold, with BM = 32 twice (a third of the rows of 192 or
    // 224, which would fit, measured no difference)
    constexpr int NB = BM > 160 || (BM == 32 && BN == 256) ? 2 : 3, NA = BM > 160 ? 2 : 3;
    constexpr int NF = BN / 64;                     // 16-row weight operands per wavefront (wavefront wn: weight rows 16 NF wn ..)
    constexpr int NCB = BN / 32;                    // copy instructions of the weights per copying wavefront and stage
    constexpr int kStageA = BM * 128, kStageB = BN * 128, kStages = NA * kStageA + NB * kStageB;
    constexpr int kOffB = NA * kStageA;             // all stages of the routed rows, then the weights': read offsets fit an instruction's 16 bits
    static_assert(kStages <= (BM == 32 ? kMoeFewLdsBytes : kMoeLdsBytes), "stages exceed the workgroup's LDS");
    constexpr int NCA = BM / 32;                    // copy instructions of the routed rows per copying wavefront and stage
    constexpr int MB = BM / 32;                     // 16-row blocks of routed rows per wavefront
    constexpr int kCopies = NCA + NCB;              // vmem operations per copying wavefront and stage
    // s_waitcnt immediate for vmcnt(n), lgkmcnt(0): vmcnt's low four bits, then its two high bits at 14
    constexpr auto vm = [](int n) constexpr { return 0x0070 | (n & 15) | ((n >> 4) << 14); };

    // (the thread's number is made opaque here and in front of the epilogue: the compiler would compute what the
    // codes for all tile sizes have in common, and the addresses of the epilogue, ahead of the loops, and spill there)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave & 3, wm = wave >> 2;
    int quad = lane >> 4;
    const int w_row0 = 16 * MB * wm;                // first routed row of the wavefront
    // Whether the weights of a stage are overwritten as soon as every wavefront has them in registers, behind a second
    // barrier in the stage: they are then copied NB stages ahead instead of NB - 1.  With two stages always; with three
    // only where there is a workgroup per CU at most, whose stages wait for the latency of memory, and not with 64 or 128
    // rows (128: whole call, us, with and without, 12 experts of 2944 x 1152, 67 rows each 52.1 / 50.3, 4 of 4096 x 1408, 100 rows
    // 56.0 / 54.3, 200 rows in two tiles 59.4 / 60.6)
    constexpr bool kCanBeEarly = NB == 2 || BM == 160 || BM == 32;
    const bool early = NB == 2 || (kCanBeEarly && few);

    const int KB = UP ? p.H : p.I;                  // bytes (= elements) per row of both operands
    const int nK = KB >> 7;
    const unsigned lds_base = (unsigned)(size_t)LDS_PTR(char, smem);

    // ---- copies: wavefronts 0-3 (one per SIMD) issue them: per stage instructions c + 4 n of the
    // routed rows (n < NCA) and of the weights (n < NCB), behind its first operand reads: spread over the stage's products
    // they measured up to 6 % slower (they have less of the stage left to land in).  Wavefronts 4-7 fetch the row scales.
    // (An L2 warm-up by these, as in the bf16 GEMM, was tried and is harmful here: an XCD's L2 holds
    // 128 KB per CU, less than the LDS stages already in flight, so lines touched early are evicted before the copies
    // ask for them.) ----
    const bool copier = wave < 4;
    const int c4 = wave & 3;
    unsigned a_off[NCA], b_off[NCB];              // 32 bits: an activation matrix, and an expert's weights, stay under 4 GiB
    auto copy_offsets = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NCA; ++n) {
            const int i = c4 + 4 * n;
            const int r = min(kt_dma_row(i, lane), rows - 1);         // rows past the tile re-read its last row
            const int src = UP ? p.sorted_tok[row0 + r] : row0 + r;
            unsigned row = (unsigned)src * (unsigned)KB;
            asm("" : "+v"(row));                    // the sum in one register: a multiply-add would be kept as 64 bits
            a_off[n] = row + 16u * (unsigned)kt_dma_chunk(i, lane);
        }
        unsigned row = (unsigned)kt_dma_row(c4, lane) * (unsigned)KB;
        asm("" : "+v"(row));
#pragma unroll
        for (int n = 0; n < NCB; ++n) {
            // first weight row of copies n of the four copying wavefronts, behind that of copies 0: 32 rows of the tile each
            const int rows_on = UP ? (n & 1) * p.I + 32 * (n >> 1) : (nt * BN + 32 * n < p.H ? 32 * n : 0);   // rows past H: others again
            b_off[n] = row + (unsigned)rows_on * (unsigned)KB + 16u * (unsigned)kt_dma_chunk(c4, lane);
        }
    };
    const char* const a_base = UP ? (const char*)p.xq : (const char*)p.aq;
    const char* const b_base = UP ? (const char*)(p.w13 + ((size_t)e * 2 * (size_t)p.I + (size_t)nt * 128) * (size_t)p.H)
                                  : (const char*)(p.w2 + ((size_t)e * (size_t)p.H + (size_t)nt * BN) * (size_t)p.I);
    const unsigned lds_copy_base = lds_base + c4 * 1024;
    // copy instruction n of stage U into LDS stage s: NCA of the routed rows, then NCB of the weights
    auto dma_part = [&](int U, int s, auto nc) __attribute__((always_inline)) {
        constexpr int n = decltype(nc)::value;
        if constexpr (n < NCA) dma_to_lds_16B<n * 4096>(a_base + (size_t)U * 128, a_off[n], lds_copy_base + s * kStageA);
        else dma_to_lds_16B<kOffB + (n - NCA) * 4096>(b_base + (size_t)U * 128, b_off[n - NCA], lds_copy_base + s * kStageB);
    };
    auto dma_rows = [&](int U, int s) __attribute__((always_inline)) {
        static_for<0, NCA>([&](auto n) __attribute__((always_inline)) { dma_part(U, s, n); });
    };
    auto dma_weights = [&](int U, int s) __attribute__((always_inline)) {
        static_for<NCA, kCopies>([&](auto n) __attribute__((always_inline)) { dma_part(U, s, n); });
    };

    // ---- scales: what the products of stage U are multiplied by, row scale x weight block scale, is worked out once per
    // row and weight block and left in LDS, [U % 2][weight block][row], one stage ahead.  Thread 256 + m does it for row m; it
    // loads the row scales of four stages at once: a row's scales lie 4 nK bytes from the next row's, so every load
    // instruction touches a cache line per row however little it takes of it.  (Copied to LDS a dword per row and stage
    // they were a third of all the lines the CU asked for.)  The weight block scales of all stages go to a table in LDS, which
    // the barrier of stage 0 makes visible; stage 0 takes its own two from memory. ----
    const LdsFloat slot = BM > 160 ? (LdsFloat)(smem + kStages) : scales;
    static_assert(BM > 160 ? kStages + 2 * 2 * BM * 4 <= kMoeLdsBytes : 2 * 2 * BM * 4 <= kMoeScaleBytes, "no room for the scales");
    typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_any;
    const float* s_src = nullptr;
    unsigned slot_at = 0;                           // LDS address of this thread's row in slot
    auto put_scales = [&](int U, float s, float sb0, float sb1) __attribute__((always_inline)) {
        if (tid - 256 < BM) {
            unsigned at = slot_at + (U & 1) * (8 * BM);
            asm("" : "+v"(at));                     // (one address, and one store of both)
            *LDS_PTR(float, (size_t)at) = s * sb0;
            *LDS_PTR(float, (size_t)(at + 4 * BM)) = s * sb1;
        }
    };
    auto sb_src = [&](int which) __attribute__((always_inline)) -> const float* {         // weight block 0 or 1 of the tile
        if (UP) return p.s13 + ((size_t)e * 2 * (p.I >> 7) + (which ? (p.I >> 7) : 0) + nt) * nK;   // gate rows, up rows of block nt
        return p.s2 + ((size_t)e * (p.H >> 7) + min(BN == 256 ? 2 * nt + which : nt, (p.H >> 7) - 1)) * nK;
    };

    // ---- per-lane LDS read addresses (stage 0): the K = 128 operand is 32 bytes of a 16-row block per lane, chunks quad and
    // quad + 4 (any order of k will do that both operands share).  A 16-byte read is served in four parts, the first of
    // which are lanes 0-3, 12-15 and 20-27: with chunks 2 quad and 2 quad + 1 the rows of two quads met in the same banks. ----
    unsigned a_addr[2], b_addr[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        a_addr[q] = lds_base + kt_offset(w_row0 + (lane & 15), quad + 4 * q);
        b_addr[q] = lds_base + kOffB + kt_offset(16 * NF * wn + (lane & 15), quad + 4 * q);
    }
    // weight block of a wavefront's operands: UP the gate block for the first half of them and the up block for the rest
    const LdsFloat my_slot = slot + (UP || BN == 128 ? 0 : wn >> 1) * BM + w_row0 + (lane & 15);
    auto frag = [&](unsigned addr0, unsigned addr1, int imm) __attribute__((always_inline)) -> i32x8 {
        const i32x4 lo = *LDS_PTR(i32x4, (size_t)(addr0 + imm));
        const i32x4 hi = *LDS_PTR(i32x4, (size_t)(addr1 + imm));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    f32x4 acc[NF][MB];
#pragma unroll
    for (int in = 0; in < NF; ++in)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[in][mb] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

    auto barrier = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- down product: where each row goes.  A row that is the only local slot of its token is that token's
    // whole sum and is written to y directly.  The lookup (row -> token -> its slots -> weight: three dependent
    // loads) is done by the wavefronts that do not copy, thread 256 + m for row m, while stage 0 is on its way; token and
    // weight are handed over through LDS once the stage buffers are free, after the loop.  Slots are loaded by eights, as one
    // by one they are a chain of KTOP round trips, and looped over, as 16 of them unrolled are 1.4 KB of code, whose
    // fetching took 0.4 us of a down product of 5.  (What an eight reads past the token's slots is the next token's, or the
    // workspace's next part, and not looked at.) ----
    int look_tok = -1;
    float look_w = 0.0f;
    auto look_up = [&](int t) __attribute__((always_inline)) {
        const int m = tid - 256;
        if (m < rows) {
            typedef __attribute__((ext_vector_type(4), aligned(4))) int i32x4_any;
            const int* const pos = p.pos + t * p.KTOP;
            int nlocal = 0, slot = 0;
            for (int k0 = 0; k0 < p.KTOP; k0 += 8) {
                const i32x4_any lo = *(const i32x4_any*)(pos + k0), hi = *(const i32x4_any*)(pos + k0 + 4);
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    if (k0 + k >= p.KTOP) break;
                    const int at = k < 4 ? lo[k & 3] : hi[k & 3];
                    nlocal += at >= 0 ? 1 : 0;
                    if (at == row0 + m) slot = k0 + k;
                }
            }
            if (nlocal == 1) { look_tok = t; look_w = p.wts[t * p.KTOP + slot]; }
        }
    };

    // ---- main loop.  It is instantiated for either role, so that no wait for a row scale, a load into registers, comes to
    // stand where a copying wavefront passes: it would wait for its copies. ----
    auto main_loop = [&](auto role) __attribute__((always_inline)) {
        constexpr bool COPIER = decltype(role)::value;
        f32x4 now, later;                                          // row scales of the next stages (the first one's in element 0), and of the four after them
        if constexpr (COPIER) {                                    // one to three stages in flight
            copy_offsets();
            __builtin_amdgcn_s_waitcnt(0x0F70);                    // vmcnt(0), known to the compiler: no wait for an earlier load inside the loop
            dma_rows(0, 0);
            dma_weights(0, 0);
            if (1 < nK) { if (NA > 2) dma_rows(1, 1); dma_weights(1, 1); }
            if (NB > 2 && early && 2 < nK) dma_weights(2, 2);
        } else {
            // Two round trips to memory, what depends on no other load and then what depends on the row's token: this chain, and
            // not the copies, is what stage 0 waits for.  (Four round trips, with the offsets of copies they do not issue and the
            // table ahead of the row scales, and a barrier in front of the copies of stage 1, took 0.3 us more.)
            slot_at = (unsigned)(size_t)slot + 4 * (tid - 256);
            const int r = min(tid - 256, rows - 1), i = min(tid - 256, 2 * nK - 1), which = i >= nK ? 1 : 0;
            const int t = p.sorted_tok[row0 + r];
            const float sb = sb_src(which)[i - which * nK], sb0 = *sb_src(0), sb1 = *sb_src(1);
            s_src = (UP ? p.xs : p.as) + (size_t)(UP ? t : row0 + r) * (size_t)nK;
            now = *(const f32x4_any*)s_src;
            later = *(const f32x4_any*)(s_src + (nK > 4 ? 4 : 0));
            if (tid - 256 < 2 * nK) sb_tab[which * kMoeMaxKB + i - which * nK] = sb;             // (2 nK <= 256)
            if constexpr (!UP) look_up(t);
            put_scales(0, now[0], sb0, sb1);
            now = __builtin_shufflevector(now, now, 1, 2, 3, 3);
        }

        // Behind which product of a stage the next stage's scales are stored: as operand reads come back in order, a store among
        // them holds up the products behind it, which a stage of few products cannot hide (BM = 64, gate/up of 8 experts of
        // 1024 x 512: 9.7 us behind the second product, 9.1 in front of the last); larger ones have the time, and the barrier
        // would wait for a late store (BM = 128, 12 of 2944 x 1152: 26.4 / 27.3)
        constexpr int kPutAt = MB <= 2 && MB * NF >= 4 ? MB * NF - 2 : 1;

        // One stage: a stream of NF products per block of 16 rows.  A product's four results are multiplied by their scale and
        // added up two products later, in the shadow of the next one; operands are read one block ahead; the order is pinned.
        int sa = 0, sb = 0;                                        // LDS stages of U
        for (int U = 0;;) {
            // stage U has landed once no more is outstanding than what was issued after it: NB - 1 stages of weights if they are
            // copied early, else one less, and the rows issued with them, towards the end fewer
            if constexpr (!COPIER) __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0): no copy of its own in flight
            else if (NA == NB && early && U + NB - 1 < nK) __builtin_amdgcn_s_waitcnt(vm((NB - 1) * NCB + (NB - 2) * NCA));
            else if (NA > 2 && U + 1 < nK) __builtin_amdgcn_s_waitcnt(vm(NCB + NCA));
            else __builtin_amdgcn_s_waitcnt(vm(0));
            asm volatile("" ::: "memory");
            barrier();                                             // stage U visible; stage U-1's buffer is free
            const LdsFloat f_row = my_slot + (U & 1) * (2 * BM);
            i32x8 fb[NF], fa[2];
            float f0[2], f1[2];
            f32x4 part[4];
            float sb0 = 0.0f, sb1 = 0.0f;                          // weight block scales of stage U + 1 (after the last stage, ones that nobody reads)
            auto read_block = [&](auto mb) __attribute__((always_inline)) {
                constexpr int set = decltype(mb)::value & 1;
                fa[set] = frag(a_addr[0], a_addr[1], mb.value * 2048);
                f0[set] = f_row[16 * mb.value];
                f1[set] = UP ? f_row[BM + 16 * mb.value] : f0[set];
            };
            auto add = [&](auto ic) __attribute__((always_inline)) {         // product i of the stage: operand i % NF, block i / NF
                constexpr int i = decltype(ic)::value;
                if constexpr (i >= 0) {
                    const float f = UP && i % NF >= NF / 2 ? f1[(i / NF) & 1] : f0[(i / NF) & 1];
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[i % NF][i / NF][r] = fmaf(part[i & 3][r], f, acc[i % NF][i / NF][r]);
                    asm volatile("" : "+v"(acc[i % NF][i / NF]));           // here: sums are else moved behind the branches around the copies, to the end
                }
            };
            auto block = [&](auto mbc) __attribute__((always_inline)) {
                constexpr int mb = decltype(mbc)::value;
                static_for<0, NF>([&](auto in) __attribute__((always_inline)) {
                    constexpr int i = mb * NF + in.value;
                    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                    part[i & 3] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fb[in.value], fa[mb & 1], zero, 0, 0, 0, 0, 0, 0);   // (scale operands 0: the plain product)
                    __builtin_amdgcn_sched_barrier(0);
                    add(IntC<i - 2>{});
                    // (the other operand set is free once the sums of the block before have taken its scales)
                    if constexpr (in.value == (NF > 2 ? 1 : NF - 1) && mb + 1 < MB) read_block(IntC<mb + 1>{});
                    if constexpr (kCanBeEarly && i == NF - 1) {
                        if (early) {                               // uniform
                            barrier();                             // every wavefront has its weights: their buffer is free
                            if constexpr (COPIER) if (U + NB < nK) dma_weights(U + NB, sb);
                        }
                    }
                    if constexpr (!COPIER && i == kPutAt) {
                        // (a load comes back behind the copies that its CU issued before it, those of the next stages: four
                        // stages ahead of its first use it holds nothing up, one stage ahead everything.  What the last group
                        // has read past the row is not used: the row after it, or the workspace's next part)
                        if (((U + 1) & 3) == 0) {
                            now = later;
                            asm volatile("" : "+v"(now) :: "memory");      // the load below goes where `later` was
                            if (U + 5 < nK) later = *(const f32x4_any*)(s_src + U + 5);
                        }
                        put_scales(U + 1, now[0], sb0, sb1);
                        now = __builtin_shufflevector(now, now, 1, 2, 3, 3);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            };
            if constexpr (!COPIER) { const int next = min(U + 1, nK - 1); sb0 = sb_tab[next]; sb1 = sb_tab[kMoeMaxKB + next]; }
            fb[0] = frag(b_addr[0], b_addr[1], 0);
            read_block(IntC<0>{});
            static_for<1, NF>([&](auto in) __attribute__((always_inline)) { fb[in.value] = frag(b_addr[0], b_addr[1], in.value * 2048); });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (COPIER) {
                if (U + NA - 1 < nK) dma_rows(U + NA - 1, sa == 0 ? NA - 1 : sa - 1);
                if (!early && U + NB - 1 < nK) dma_weights(U + NB - 1, sb == 0 ? NB - 1 : sb - 1);
            }
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, MB>(block);
            add(IntC<MB * NF - 2>{});
            add(IntC<MB * NF - 1>{});
            if (++U >= nK) break;
            const int wrap_a = sa + 1 == NA ? NA : 0, wrap_b = sb + 1 == NB ? NB : 0;
            sa += 1 - wrap_a;
            sb += 1 - wrap_b;
#pragma unroll
            for (int q = 0; q < 2; ++q) { a_addr[q] += (1 - wrap_a) * kStageA; b_addr[q] += (1 - wrap_b) * kStageB; }
        }
    };
    if (copier) main_loop(IntC<1>{}); else main_loop(IntC<0>{});

    // ---- epilogue: result layout of a lane: register r of operand `in`, block mb is weight row 16 in + 4 quad + r of the wavefront's
    // 16 NF, routed row w_row0 + 16 mb + lane%16
    asm volatile("" : "+v"(lane));
    quad = lane >> 4;
    if constexpr (UP) {
        // SiLU gate, then quant128 over the tile's 128 columns of each routed row
        float amax[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            amax[mb] = 0.0f;
#pragma unroll
            for (int in = 0; in < 2; ++in)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float g = acc[in][mb][r];
                    acc[in][mb][r] = g / (1.0f + __expf(-g)) * acc[in + 2][mb][r];
                    amax[mb] = fmaxf(amax[mb], fabsf(acc[in][mb][r]));
                }
            // across the four quarters of the wavefront
            amax[mb] = fmaxf(amax[mb], __shfl_xor(amax[mb], 16));
            amax[mb] = fmaxf(amax[mb], __shfl_xor(amax[mb], 32));
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        barrier();                                             // every wavefront is done with the stage buffers
        const LdsFloat ex = (LdsFloat)smem;                        // [wm][mb][wn][16]
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
            if (quad == 0) ex[((wm * MB + mb) * 4 + wn) * 16 + lane] = amax[mb];
        __builtin_amdgcn_s_waitcnt(0xC07F);
        barrier();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            float am = amax[mb];
#pragma unroll
            for (int w = 0; w < 4; ++w) am = fmaxf(am, ex[((wm * MB + mb) * 4 + w) * 16 + (lane & 15)]);
            const float scale = quant_scale(am);
            const float inv = 1.0f / scale;
            const int m = w_row0 + 16 * mb + (lane & 15);
            if (m < rows) {
                uint8_t* const dst = p.aq + (size_t)(row0 + m) * p.I + nt * 128 + 32 * wn + 4 * quad;
#pragma unroll
                for (int in = 0; in < 2; ++in)
                    *(unsigned*)(dst + 16 * in) = quant_pack4(acc[in][mb][0], acc[in][mb][1], acc[in][mb][2], acc[in][mb][3], inv);
                if (wn == 0 && quad == 0) p.as[(size_t)(row0 + m) * (p.I >> 7) + nt] = scale;
            }
        }
    } else {
        // A row that is the only local slot of its token is that token's whole sum: weight * row, rounded once
        // to bf16, goes to y directly (bit for bit what the combine step computes from the fp32 row) and the
        // fp32 row is neither written nor read again.  Other rows go to the workspace for moe_combine.
        static_assert(BM <= 256, "one lookup thread per row");
        __builtin_amdgcn_s_waitcnt(0xC07F);
        barrier();                                             // every wavefront is done with the stage buffers
        const LdsFloat hand = (LdsFloat)smem;                  // [row][token bits, weight]
        if (tid >= 256 && tid - 256 < BM) { hand[2 * (tid - 256)] = __int_as_float(look_tok); hand[2 * (tid - 256) + 1] = look_w; }
        __builtin_amdgcn_s_waitcnt(0xC07F);
        barrier();
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = w_row0 + 16 * mb + (lane & 15);
            if (m < rows) {
                const int dst = __float_as_int(hand[2 * m]);
                const float w = hand[2 * m + 1];
#pragma unroll
                for (int in = 0; in < NF; ++in) {
                    const int c = nt * BN + 16 * NF * wn + 16 * in + 4 * quad;
                    if (c < p.H) {
                        const f32x4 v = acc[in][mb];
                        if (dst >= 0) {
                            const bf16x4 out = {(__bf16)fmaf(w, v[0], 0.0f), (__bf16)fmaf(w, v[1], 0.0f), (__bf16)fmaf(w, v[2], 0.0f), (__bf16)fmaf(w, v[3], 0.0f)};   // as moe_combine: 0 + w * v
                            *(bf16x4*)(p.y + (size_t)dst * p.H + c) = out;
                        } else {
                            *(f32x4*)(p.o + (size_t)(row0 + m) * p.H + c) = v;
                        }
                    }
                }
            }
        }
    }
}

// Workgroup -> row tile and column tile; false if there is none for it (uniform, before any barrier).  The grid has
// max_tiles * NT workgroups (a multiple of 8), of which ntiles * NT are live; XCD x (= blockIdx % 8) takes the x-th eighth
// of the live logical ids in order, so the workgroups resident on an XCD are neighbours.  Logical order: expert by expert;
// inside an expert column tile by column tile, the expert's row tiles innermost: neighbours share their weight tile (same
// nt) or their routed rows (same row tile), which the XCD's L2 then fetches once.
struct MoeTile { int e, row0, rows, nt; };
__device__ __forceinline__ bool moe_tile_of(const MoeParams& p, int NT, int live, int bm, MoeTile& t) {
    const int per_xcd = (live + 7) >> 3, bid = blockIdx.x, logical = (bid & 7) * per_xcd + (bid >> 3);
    if ((bid >> 3) >= per_xcd || logical >= live) return false;
    const MoeTileRec rec = p.tile_rec[logical / NT];             // the expert whose block of ids holds `logical`
    const int cnt = moe_tiles(rec.rows, bm);                      // its row tiles
    const int off = logical - rec.first * NT;                     // in [0, cnt * NT)
    const int nt = off / cnt, j = off - nt * cnt;                 // column tile, row tile within the expert
    const int begin = moe_tile_begin(rec.rows, cnt, j, bm);
    t.e = __builtin_amdgcn_readfirstlane(rec.expert);
    t.row0 = __builtin_amdgcn_readfirstlane(rec.row0 + begin);
    t.rows = __builtin_amdgcn_readfirstlane(moe_tile_begin(rec.rows, cnt, j + 1, bm) - begin);
    t.nt = __builtin_amdgcn_readfirstlane(nt);
    return true;
}

// Kernel for few rows per expert (MoeParams::few): tiles of 32 rows in two stages of weights and three of rows (three of either
// where the column tiles are halved), so that two workgroups share a CU and one starts and ends while the other streams.  Reading the weights bounds it:
// gate/up / down, us, against the 64-row code with one workgroup per CU: 40 tokens of (2048 x 1408, 64 experts) 68.7 / 32.2
// -> 63.1 / 28.7, 60 of (2048 x 768, 128 experts) 71.3 / 40.0 -> 66.4 / 31.8.  An expert with more than 32 rows is several
// tiles, neighbours in the order of workgroups, so that its weights come from HBM once.  (As one tile of two passes it was the last to
// end: 64 tokens on 16 experts of 6144 x 2048, most of them on one, 96 us for the call against 55.)
template <bool UP>
__global__ __launch_bounds__(512, 4) void moe_gemm_few(MoeParams p) {
    constexpr int BM = 32;
    __shared__ __attribute__((aligned(16))) char smem[kMoeFewLdsBytes];
    __shared__ __attribute__((aligned(16))) float scales[2 * 2 * BM];
    static_assert(2 * (kMoeFewLdsBytes + 2 * 2 * BM * 4 + 2 * kMoeMaxKB * 4) <= 160 * 1024, "LDS budget");
    __shared__ float sb_tab[2 * kMoeMaxKB];
    const int ntl = p.ntiles[0], bm = p.ntiles[1];
    // half column tiles as in moe_gemm, although a CU holds two workgroups here.  Down product, us, at other limits: 64 tiles, 84 wide
    // ones of (7168 x 2048) 10.5 -> 14.2, 112 of (4096 x 14336) 70 -> 97; 256, 140 of the former 14.7 -> 17.2, 224 20.2 -> 19.4
    const bool narrow = !UP && p.dn_narrow_ok && ntl * ((p.H + kMoeBN - 1) / kMoeBN) <= 128;
    const int NT = UP ? (p.I >> 7) : narrow ? (p.H >> 7) : (p.H + kMoeBN - 1) / kMoeBN;
    MoeTile t;
    if (!moe_tile_of(p, NT, ntl * NT, bm, t)) return;
    const LdsChar tiles = LDS_PTR(char, smem);
    const LdsFloat sa = LDS_PTR(float, scales), sb = LDS_PTR(float, sb_tab);
    if constexpr (!UP) {
        if (narrow) { moe_gemm_tile<false, BM, 128>(p, t.e, t.row0, t.rows, t.nt, true, tiles, sa, sb); return; }
    }
    moe_gemm_tile<UP, BM, 256>(p, t.e, t.row0, t.rows, t.nt, true, tiles, sa, sb);
}

// Kernel: maps the workgroup to its (row tile, column tile) and runs the tile code that fits the tile's rows.
template <bool UP>
__global__ __launch_bounds__(512, 1) void moe_gemm(MoeParams p) {
    __shared__ __attribute__((aligned(16))) char smem[kMoeLdsBytes];
    __shared__ __attribute__((aligned(16))) float scales[kMoeScaleBytes / 4];
    static_assert(kMoeLdsBytes + kMoeScaleBytes + 2 * kMoeMaxKB * 4 <= 160 * 1024, "LDS budget");
    __shared__ float sb_tab[2 * kMoeMaxKB];          // weight block scale of the tile's two 128-row blocks and every stage

    // Down product: column tiles of 256 weight rows, or of 128 when the wide ones would fill half the chip at most (few
    // experts in use, or a small H: 8 experts of 4096 x 14336 make 128 wide tiles).  The host sizes the grid for the
    // narrow tiles when the problem is small enough for that to happen (p.dn_narrow_ok); the choice itself needs the
    // number of row tiles, known only here.  Narrow against wide, us: 64 wide tiles (4 experts of 4096 x 1408, 100 rows)
    // 12.0 / 16.8, 128 (8 of 4096 x 14336, 130 rows) 122 / 196, (8 of 1024 x 512, 1000 rows) 15.9 / 20.5; with more than
    // 128 the narrow ones run two rounds: 144 (12 of 2944 x 1152, 100 rows) 21.2 / 17.0, 192 (8 of 1024 x 512, 700 rows)
    // 15.3 / 13.2; with more than 256 they are 3-15 % slower.
    const int ntl = p.ntiles[0], bm = p.ntiles[1];
    const bool narrow = !UP && p.dn_narrow_ok && ntl * ((p.H + kMoeBN - 1) / kMoeBN) <= 128;
    const int NT = UP ? (p.I >> 7) : narrow ? (p.H >> 7) : (p.H + kMoeBN - 1) / kMoeBN;
    const int live = ntl * NT;
    MoeTile t;
    if (!moe_tile_of(p, NT, live, bm, t)) return;
    const int e = t.e, row0 = t.row0, rows = t.rows, nt = t.nt;
    const bool few = live <= 256;
    const LdsChar tiles = LDS_PTR(char, smem);
    const LdsFloat sa = LDS_PTR(float, scales), sb = LDS_PTR(float, sb_tab);
    if constexpr (!UP) {
        if (narrow) {
            if (rows > 224) moe_gemm_tile<false, 256, 128>(p, e, row0, rows, nt, few, tiles, sa, sb);
            else if (rows > 192) moe_gemm_tile<false, 224, 128>(p, e, row0, rows, nt, few, tiles, sa, sb);
            else if (rows > 160) moe_gemm_tile<false, 192, 128>(p, e, row0, rows, nt, few, tiles, sa, sb);
            else if (rows > 128) moe_gemm_tile<false, 160, 128>(p, e, row0, rows, nt, few, tiles, sa, sb);
            else if (rows > 64) moe_gemm_tile<false, 128, 128>(p, e, row0, rows, nt, few, tiles, sa, sb);
            else moe_gemm_tile<false, 64, 128>(p, e, row0, rows, nt, few, tiles, sa, sb);
            return;
        }
    }
    if (rows > 224) moe_gemm_tile<UP, 256, 256>(p, e, row0, rows, nt, few, tiles, sa, sb);
    else if (rows > 192) moe_gemm_tile<UP, 224, 256>(p, e, row0, rows, nt, few, tiles, sa, sb);
    else if (rows > 160) moe_gemm_tile<UP, 192, 256>(p, e, row0, rows, nt, few, tiles, sa, sb);
    else if (rows > 128) moe_gemm_tile<UP, 160, 256>(p, e, row0, rows, nt, few, tiles, sa, sb);
    else if (rows > 64) moe_gemm_tile<UP, 128, 256>(p, e, row0, rows, nt, few, tiles, sa, sb);
    else moe_gemm_tile<UP, 64, 256>(p, e, row0, rows, nt, few, tiles, sa, sb);
}

// ------------------------------------------------------------------------------------
// Combine: y[t][c] = sum over local slots k (ascending) of wts[t][k] * o[pos[t][k]][c], bf16.  Tokens with exactly
// one local slot were written by the down product; those with none get zeros.
// What bounds it: y, mostly zeros where the experts are spread over ranks, and the rows of o.  A wavefront takes a token,
// or one of `segs` interleaved parts of its columns where there are few tokens: the slots are one load of a lane each
// (read one after the other they were a chain of KTOP round trips in each of 65536 short workgroups: 58 us for
// T16384 H7168 with 137 MB to write and 75 MB to read, now 45), and up to four rows of o are in flight at once.
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void moe_combine(MoeParams p, int segs) {
    const int lane = threadIdx.x & 63, item = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = item / segs, seg = item - t * segs;
    if (t >= p.T) return;
    const int pos = lane < p.KTOP ? p.pos[t * p.KTOP + lane] : -1;
    const float wt = lane < p.KTOP ? p.wts[t * p.KTOP + lane] : 0.0f;
    const unsigned long long local = __builtin_amdgcn_ballot_w64(pos >= 0);
    const int nlocal = __popcll(local);
    if (nlocal == 1) return;
    __bf16* const y = p.y + (size_t)t * p.H;
    for (int c = seg * 512 + lane * 8; c < p.H; c += segs * 512) {
        float acc[8] = {};
        for (unsigned long long left = local; left != 0;) {
            constexpr int NR = 4;
            f32x4 a[NR], b[NR];
            float w[NR];
            int n = 0;
#pragma unroll
            for (int j = 0; j < NR; ++j) {
                if (left != 0) {                              // uniform
                    const int k = __builtin_ctzll(left);
                    left &= left - 1;
                    w[j] = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(wt), k));
                    const float* const o = p.o + (size_t)__builtin_amdgcn_readlane(pos, k) * p.H + c;
                    a[j] = *(const f32x4*)o;
                    b[j] = *(const f32x4*)(o + 4);
                    n = j + 1;
                }
            }
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (j < n) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) { acc[i] = fmaf(w[j], a[j][i], acc[i]); acc[4 + i] = fmaf(w[j], b[j][i], acc[4 + i]); }
                }
        }
        bf16x8 out;
#pragma unroll
        for (int i = 0; i < 8; ++i) out[i] = (__bf16)acc[i];
        *(bf16x8*)(y + c) = out;
    }
}

}  // namespace

// Scratch memory for callers that cannot allocate (graph capture, tight serving loops): one array per GPU, part
// of the code object, alive until the process ends.  In host code the array's NAME is only a handle for the
// symbol lookup below, never an address: every use of its memory goes through the pointer the lookup returned
// for the device at hand (each GPU holds its own copy at its own address).
static __device__ __align__(256) unsigned char moe_scratch_array[kMoeStaticScratchBytes];

void* moe_static_scratch(size_t* bytes) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* ptrs[kMaxDevices] = {};
    if (bytes) *bytes = kMoeStaticScratchBytes;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(moe_scratch_array)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        ptrs[dev] = ptr;
    }
    return ptrs[dev];
}

int moe_launch(const MoeParams& p, int first, int last, hipStream_t stream) {
    auto on = [&](int stage) { return first <= stage && stage <= last; };
    const long long items = (long long)p.T * ((p.H / 128 + kMoeQuantGroups - 1) / kMoeQuantGroups);   // quantization: kMoeQuantGroups groups of a token per 32 lanes
    if (on(0) || on(1))
        hipLaunchKernelGGL(moe_prepare, dim3(1 + (on(1) ? (unsigned)((items + 31) / 32) : 0u)), dim3(1024), 0, stream, p,
                           (on(0) ? 1 : 0) | (on(1) ? 2 : 0));
    auto grid8 = [](long long n) { return dim3((unsigned)((n + 7) / 8 * 8)); };   // the tile order wants a multiple of 8
    const dim3 g_up = grid8((long long)p.max_tiles * (p.I / 128)),
               g_dn = grid8((long long)p.max_tiles * (p.dn_narrow_ok ? p.H / 128 : (p.H + kMoeBN - 1) / kMoeBN));
    if (p.few) {
        if (on(2)) hipLaunchKernelGGL((moe_gemm_few<true>), g_up, dim3(512), 0, stream, p);
        if (on(3)) hipLaunchKernelGGL((moe_gemm_few<false>), g_dn, dim3(512), 0, stream, p);
    } else {
        if (on(2)) hipLaunchKernelGGL((moe_gemm<true>), g_up, dim3(512), 0, stream, p);
        if (on(3)) hipLaunchKernelGGL((moe_gemm<false>), g_dn, dim3(512), 0, stream, p);
    }
    if (on(4)) {
        // parts of a token's columns: enough wavefronts for the chip (8192 slots) down to one pass of 512 columns each
        const int most = (p.H + 511) / 512, want = (8192 + p.T - 1) / p.T, segs = want < most ? want : most;
        hipLaunchKernelGGL(moe_combine, dim3((unsigned)(((long long)p.T * segs + 3) / 4)), dim3(256), 0, stream, p, segs);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}
