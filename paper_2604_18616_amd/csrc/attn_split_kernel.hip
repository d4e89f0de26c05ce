// Attention forward for few query rows or few heads (decoding, speculated tokens, chunks) on gfx950: the keys, not the
// query rows, are what there is to spread over the chip.
//
// The query rows that share a kv head (g = Hq / Hkv heads x Sq positions) are packed into 32-row blocks, one block
// per wavefront column of the MFMA, and the keys of that kv head are cut twice: over `splits` workgroups, and inside
// a workgroup over KG groups of wavefronts.  Each group streams its own 32-key tiles HBM -> LDS into two private
// stages and keeps its own running maximum, sum and O; the groups of a workgroup are merged through LDS, the
// workgroups of a row by attn_split_combine from fp32 rows in the caller's workspace (with one workgroup per row
// block the result goes straight to O).
//
// What bounds it: reading K and V once.  A workgroup of 4 wavefronts keeps 64-128 KB of copies in flight per CU,
// and with one key group per wavefront (RB = 1) there is no barrier in the loop at all: a wavefront only waits for
// its own copies.  Measured at D = 128, B Hq Hkv Sq Sk, against a 128-row workgroup per query head: 32 32 8 1 4096:
// 295 -> 102 us (5.3 TB/s of K and V); 1 32 8 1 2000: 47.6 -> 10 us (two launches, latency); 1 8 1 4 60000: 1230 -> 15 us;
// 2 64 8 4 9001: 191 -> 20 us; 1 8 8 33 5000: 110 -> 13 us; with few long heads the cut is what fills the chip, with
// many heads that the heads of a group read K and V once instead of Hq / Hkv times.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "attn_layout.h"
#include "attn_launch.h"
#include "gfx950_prims.h"

namespace {

using namespace attn_layout;
using namespace gfx950;

constexpr int kFewSplits = 8;       // splits up to which a thread adds them up alone
constexpr int kTileKeys = 32;      // keys per tile and key group

__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }

// Query row r of a kv head's g * Sq packed rows -> offset of its head among the g, position.  The g heads of a position lie
// side by side: a 32-row block spans 32 / g positions, inside one group of 32 of them for any g, so that under the
// causal mask its rows end at nearly the same key.
struct PackedRow { int h, i; };
__device__ __forceinline__ PackedRow packed_row(int r, int g) {
    PackedRow x;
    x.i = r / g;
    x.h = r - x.i * g;
    return x;
}

template <int D> constexpr int split_pitch() { return D + 4; }          // floats per O row in the merge area: 4 consecutive floats of 32 rows land in different banks
template <int D, int RB, int NW> constexpr int split_smem_bytes() {
    constexpr int KG = NW / RB;
    constexpr int stages = KG * 2 * 2 * kTileKeys * D * 2;
    constexpr int merge = KG == 1 ? 0 : NW * kWaveRows * split_pitch<D>() * 4;
    return stages > merge ? stages : merge;
}

// RB row blocks of 32 packed query rows x KG = 4 / RB key groups.  RB = 1: a wavefront copies its own tiles.
// RB > 1: the RB wavefronts of a group share its tiles (two workgroup barriers per tile), which divides the copies
// per FLOP by RB: for more than 32 rows per kv head, where the copies L2 -> LDS are what bounds RB = 1.
template <int D, bool CAUSAL, int RB, int NW>
__global__ __launch_bounds__(NW * 64, NW == 2 ? 1 : (D == 128 && RB == 1) ? 1 : 2) void attn_fwd_split(AttnParams p, AttnSplit sp) {
    constexpr int KG = NW / RB;
    constexpr int KS = D / 16, DB = D / 32, CPR = D / 8;
    constexpr int TB = kTileKeys * D * 2;          // bytes of a K or V tile
    constexpr int RPI = dma_rows_per_inst<D>();    // rows per 1 KB copy
    constexpr int NI = TB / 1024 / RB;             // copies per wavefront, tile and matrix
    constexpr int PITCH = split_pitch<D>();

    __shared__ __attribute__((aligned(1024))) char smem[split_smem_bytes<D, RB, NW>()];
    __shared__ float sml[2][NW][kWaveRows];        // maximum and sum of every wavefront's rows
    __shared__ float s_inv[RB * kWaveRows];
    __shared__ long long s_row[RB * kWaveRows];    // where a row of the result or of the parts starts

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rb = wave % RB, kg = wave / RB;

    // Workgroup id -> (kv head of a sequence, split, row blocks).  Row blocks of one split read the same keys:
    // they are neighbours in the order of which every XCD (its own L2) takes a contiguous range.
    const int nb = gridDim.x, per_xcd = nb >> 3, bid = blockIdx.x;
    int logical = bid < per_xcd * 8 ? (bid & 7) * per_xcd + (bid >> 3) : bid;
    const int rowblk = logical % sp.row_wgs;
    logical /= sp.row_wgs;
    const int split = logical % sp.splits;
    logical /= sp.splits;
    const int hk = logical % p.Hkv, b = logical / p.Hkv;

    const int g = p.Hq / p.Hkv, Sq = p.Sq, Sk = p.Sk, R = g * Sq, shift = Sk - Sq;
    const __bf16* kh = p.k + b * p.k_sb + hk * p.k_sh;
    const __bf16* vh = p.v + b * p.v_sb + hk * p.v_sh;

    // key tiles this workgroup's rows can see, and this split's share of them
    const int first = rowblk * (RB * kWaveRows), last = min(first + RB * kWaveRows, R) - 1;
    const int lim_wg = CAUSAL ? min(Sk - 1, packed_row(last, g).i + shift) : Sk - 1;
    const int nT = lim_wg < 0 ? 0 : lim_wg / kTileKeys + 1;
    const int per = (nT + sp.splits - 1) / sp.splits;
    const int t0 = split * per, t1 = min(nT, t0 + per);

    const int r = first + rb * kWaveRows + (lane & 31);
    const PackedRow row = packed_row(min(r, R - 1), g);
    const int lim = CAUSAL ? min(Sk - 1, row.i + shift) : Sk - 1;
    // the last key any row of this wavefront sees: later tiles are left out, so that V behind the mask (0 * inf is NaN)
    // reaches no row from further away than the mask's own tile
    const int lim_wave = CAUSAL ? min(Sk - 1, packed_row(min(first + rb * kWaveRows + kWaveRows, R) - 1, g).i + shift) : Sk - 1;
    const float c = p.scale_log2;

    // copies: lane offsets inside a tile (the LDS side is lane-contiguous, the swizzle is applied to the source)
    const unsigned k_rb = 2u * (unsigned)p.k_ss, v_rb = 2u * (unsigned)p.v_ss;
    const i32x4 k_rsrc = buffer_resource(kh, (unsigned)(Sk - 1) * k_rb + 2u * D);   // rows past Sk - 1 arrive as zeros
    const i32x4 v_rsrc = buffer_resource(vh, (unsigned)(Sk - 1) * v_rb + 2u * D);
    unsigned koff[NI], voff[NI];
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        const int trow = (rb + RB * n) * RPI + lane / CPR, pos = lane % CPR;
        koff[n] = (unsigned)trow * k_rb + 16u * (unsigned)(pos ^ k_swizzle<D>(trow));
        voff[n] = (unsigned)trow * v_rb + 16u * (unsigned)(pos ^ v_swizzle<D>(trow));
    }
    const unsigned lds_base = (unsigned)(size_t)LDS_PTR(char, smem) + (unsigned)kg * (4 * TB);
    const unsigned zero_off = 0;
    auto issue = [&](int t, int st) __attribute__((always_inline)) {
        const unsigned kt = (unsigned)(t * kTileKeys) * k_rb, vt = (unsigned)(t * kTileKeys) * v_rb;
#pragma unroll
        for (int n = 0; n < NI; ++n)
            dma_buf_to_lds_16B(k_rsrc, koff[n] + kt, zero_off, lds_base + st * (2 * TB) + (rb + RB * n) * 1024);
#pragma unroll
        for (int n = 0; n < NI; ++n)
            dma_buf_to_lds_16B(v_rsrc, voff[n] + vt, zero_off, lds_base + st * (2 * TB) + TB + (rb + RB * n) * 1024);
    };

    f32x16 oacc[DB];
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[i][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    // every group runs the same number of steps, so that the barriers of RB > 1 match
    const int steps = t1 > t0 ? (t1 - t0 + KG - 1) / KG : 0;
    if (t0 + kg < t1) issue(t0 + kg, 0);
    if (t0 + kg + KG < t1) issue(t0 + kg + KG, 1);
    bf16x8 qf[KS];
    {
        const __bf16* qrow = p.q + b * p.q_sb + (hk * g + row.h) * p.q_sh + (long long)row.i * p.q_ss + 8 * half;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *(const bf16x8*)(qrow + 16 * ks);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0), known to the compiler: no wait for Q inside the loop
    asm volatile("" ::: "memory");

    for (int s = 0; s < steps; ++s) {
        const int t = t0 + kg + s * KG, st = s & 1;
        if constexpr (RB > 1) { __builtin_amdgcn_sched_barrier(0); __builtin_amdgcn_s_barrier(); __builtin_amdgcn_sched_barrier(0); }
        if (t < t1 && t * kTileKeys <= lim_wave) {
            const char* const sK = smem + kg * (4 * TB) + st * (2 * TB);
            const char* const sV = sK + TB;
            f32x16 sc;
#pragma unroll
            for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const bf16x8 kf = *(const bf16x8*)(sK + k_chunk_offset<D>(qk_key_row(lane, 0), qk_chunk(lane, ks)));
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], sc, 0, 0, 0);
            }
            const int room = lim - t * kTileKeys - 4 * half;
            if (__builtin_amdgcn_ballot_w64(room < kTileKeys - 4 * half - 1) != 0) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    if (8 * (e / 4) + e % 4 > room) sc[e] = -INFINITY;
            }
            float mx = sc[0];
#pragma unroll
            for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
            mx = max_across_halves(mx);
            const float m_new = fmaxf(m_run, mx);
            const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
            const float alpha = exp2_hw((m_run - m_use) * c);
            m_run = m_new;
            const float mc = m_use * c;
            float psum = 0.f;
            unsigned pk[8];
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
                const float p0 = exp2_hw(fmaf(sc[e], c, -mc));
                const float p1 = exp2_hw(fmaf(sc[e + 1], c, -mc));
                psum += p0 + p1;
                pk[e >> 1] = pack_bf16x2(p0, p1);
            }
            l_run = l_run * alpha + psum;
            if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
                for (int i = 0; i < DB; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) oacc[i][e] *= alpha;
            }
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const u32x4 pw = {pk[4 * kk], pk[4 * kk + 1], pk[4 * kk + 2], pk[4 * kk + 3]};
                const bf16x8 pf = __builtin_bit_cast(bf16x8, pw);
#pragma unroll
                for (int dblk = 0; dblk < DB; ++dblk) {
                    const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, sV + pv_addr_offset<D>(lane, dblk, kk, 0)));
                    const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, sV + pv_addr_offset<D>(lane, dblk, kk, 1)));
                    const s16x8 vv = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
                    oacc[dblk] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vv), pf, oacc[dblk], 0, 0, 0);
                }
            }
        }
        // the stage is free once its reads have returned; then the copies of the tile after next go into it, and the
        // wait is for the tile in between
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if constexpr (RB > 1) { __builtin_amdgcn_sched_barrier(0); __builtin_amdgcn_s_barrier(); __builtin_amdgcn_sched_barrier(0); }
        if (t + 2 * KG < t1) {
            issue(t + 2 * KG, st);
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * NI) : "memory");
        } else {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
    }

    const float l_wave = sum_across_halves(l_run);
    auto row_index = [&](const PackedRow& x) __attribute__((always_inline)) {
        return ((size_t)b * p.Hq + hk * g + x.h) * (size_t)Sq + x.i;
    };
    auto o_row = [&](const PackedRow& x) __attribute__((always_inline)) {
        return p.o + b * p.o_sb + (hk * g + x.h) * p.o_sh + (long long)x.i * p.o_ss;
    };
    // four consecutive values of a row: the result, or this split's part of it
    auto put4 = [&](const PackedRow& x, int d, f32x4 v, float l) __attribute__((always_inline)) {
        if (sp.splits == 1) {
            const float inv = l > 0.f ? 1.0f / l : 0.f;
            u32x2 w;
            w[0] = pack_bf16x2(v[0] * inv, v[1] * inv);
            w[1] = pack_bf16x2(v[2] * inv, v[3] * inv);
            *(u32x2*)(o_row(x) + d) = w;
        } else {
            *(f32x4*)(sp.part + (row_index(x) * sp.splits + split) * D + d) = v;
        }
    };
    auto put_ml = [&](const PackedRow& x, float m, float l) __attribute__((always_inline)) {
        if (sp.splits == 1) {
            if (p.lse != nullptr) p.lse[row_index(x)] = l > 0.f ? m * p.scale + logf(l) : -INFINITY;
        } else {
            *(f32x2*)(sp.ml + 2 * (row_index(x) * sp.splits + split)) = f32x2{m, l};
        }
    };

    if constexpr (KG == 1) {
        if (r < R) {
#pragma unroll
            for (int dblk = 0; dblk < DB; ++dblk)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4)
                    put4(row, o_d(lane, dblk, 4 * g4),
                         f32x4{oacc[dblk][4 * g4], oacc[dblk][4 * g4 + 1], oacc[dblk][4 * g4 + 2], oacc[dblk][4 * g4 + 3]}, l_wave);
            if (half == 0) put_ml(row, m_run, l_wave);
        }
    } else {
        // merge the key groups: every wavefront scales its rows of O to the maximum over the groups and leaves them in
        // LDS; what the threads that add them up need to know about a row is worked out once per row
        if (half == 0) { sml[0][wave][lane] = m_run; sml[1][wave][lane] = l_wave; }
        __syncthreads();                                  // also: nobody reads the stages any more
        if (r < R) {
            const int rw = lane & 31;
            float m = sml[0][rb][rw], l = 0.f;
#pragma unroll
            for (int k = 1; k < KG; ++k) m = fmaxf(m, sml[0][k * RB + rb][rw]);
            const float f = m_run == -INFINITY ? 0.f : exp2_hw((m_run - m) * c);
            float* const dst = (float*)smem + (wave * kWaveRows + rw) * PITCH;
#pragma unroll
            for (int dblk = 0; dblk < DB; ++dblk)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4)
                    *(f32x4*)(dst + o_d(lane, dblk, 4 * g4)) = f32x4{oacc[dblk][4 * g4] * f, oacc[dblk][4 * g4 + 1] * f,
                                                                    oacc[dblk][4 * g4 + 2] * f, oacc[dblk][4 * g4 + 3] * f};
            if (kg == 0 && half == 0) {
#pragma unroll
                for (int k = 0; k < KG; ++k) {
                    const float mk = sml[0][k * RB + rb][rw];
                    l += sml[1][k * RB + rb][rw] * (mk == -INFINITY ? 0.f : exp2_hw((mk - m) * c));   // a NaN sum stays one
                }
                put_ml(row, m, l);
                s_inv[rb * kWaveRows + rw] = l > 0.f ? 1.0f / l : 0.f;
                s_row[rb * kWaveRows + rw] = sp.splits == 1 ? (long long)(hk * g + row.h) * p.o_sh + (long long)row.i * p.o_ss
                                                            : (long long)(row_index(row) * sp.splits + split) * D;
            }
        }
        __syncthreads();
        constexpr int QPR = D / 4;                        // groups of four values per row
#pragma unroll
        for (int j = 0; j < RB * kWaveRows * QPR / (NW * 64); ++j) {
            const int item = j * (NW * 64) + tid, rr = item / QPR, d = (item % QPR) * 4;
            if (first + rr < R) {
                const float* const src = (const float*)smem + rr * PITCH + d;   // row rr of group k: RB * 32 rows further on
                f32x4 v = *(const f32x4*)src;
#pragma unroll
                for (int k = 1; k < KG; ++k) v += *(const f32x4*)(src + k * (RB * kWaveRows * PITCH));
                if (sp.splits == 1) {
                    const float inv = s_inv[rr];
                    u32x2 w;
                    w[0] = pack_bf16x2(v[0] * inv, v[1] * inv);
                    w[1] = pack_bf16x2(v[2] * inv, v[3] * inv);
                    *(u32x2*)(p.o + b * p.o_sb + s_row[rr] + d) = w;
                } else {
                    *(f32x4*)(sp.part + s_row[rr] + d) = v;
                }
            }
        }
    }
}

// The same for few splits and many rows: D/4 threads per row, each adding up its own four columns.
template <int D>
__global__ __launch_bounds__(256) void attn_split_combine_few(AttnParams p, AttnSplit sp, unsigned rows) {
    constexpr int QPR = D / 4;
    const int S = sp.splits, d = (threadIdx.x % QPR) * 4;
    const size_t rowi = (size_t)blockIdx.x * (256 / QPR) + threadIdx.x / QPR;
    if (rowi >= rows) return;
    f32x4 v[kFewSplits];
    f32x2 ml[kFewSplits];
    float m = -INFINITY, l = 0.f;
#pragma unroll
    for (int s = 0; s < kFewSplits; ++s) {
        v[s] = s < S ? *(const f32x4*)(sp.part + (rowi * S + s) * D + d) : f32x4{0.f, 0.f, 0.f, 0.f};
        ml[s] = s < S ? *(const f32x2*)(sp.ml + 2 * (rowi * S + s)) : f32x2{-INFINITY, 0.f};
    }
#pragma unroll
    for (int s = 0; s < kFewSplits; ++s) m = fmaxf(m, ml[s][0]);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < kFewSplits; ++s) {
        const float w = ml[s][0] == -INFINITY ? 0.f : exp2_hw((ml[s][0] - m) * p.scale_log2);
        l += ml[s][1] * w;
        acc += v[s] * w;
    }
    const float inv = l > 0.f ? 1.0f / l : 0.f;
    const int i = (int)(rowi % p.Sq);
    const size_t bh = rowi / p.Sq;
    const int hq = (int)(bh % p.Hq), b = (int)(bh / p.Hq);
    u32x2 w2;
    w2[0] = pack_bf16x2(acc[0] * inv, acc[1] * inv);
    w2[1] = pack_bf16x2(acc[2] * inv, acc[3] * inv);
    *(u32x2*)(p.o + b * p.o_sb + hq * p.o_sh + (long long)i * p.o_ss + d) = w2;
    if (d == 0 && p.lse != nullptr) p.lse[rowi] = l > 0.f ? m * p.scale + logf(l) : -INFINITY;
}

// O and LSE of one query row from the parts of its splits: one workgroup per row, NS = 256 / (D/4) splits side by
// side, up to eight loads per thread in flight (the parts come from L2 or the memory-side cache: latency counts).
template <int D>
__global__ __launch_bounds__(256) void attn_split_combine(AttnParams p, AttnSplit sp) {
    constexpr int QPR = D / 4, NS = 256 / QPR, NL = 8, NM = kMaxSplits / 64;
    __shared__ float red[NS][D];
    const int tid = threadIdx.x, lane = tid & 63, sl = tid / QPR, d = (tid % QPR) * 4, S = sp.splits;
    const size_t rowi = blockIdx.x;
    const float* const part = sp.part + rowi * S * D + d;
    f32x4 v[NL];
    auto load = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int n = 0; n < NL; ++n) {
            const int s = s0 + sl + n * NS;
            v[n] = s < S ? *(const f32x4*)(part + (size_t)s * D) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    load(0);
    // weights: split 64 j + lane in w[j] of every wavefront
    float mm[NM], ll[NM], w[NM], m = -INFINITY, l = 0.f;
#pragma unroll
    for (int j = 0; j < NM; ++j) {
        const int s = 64 * j + lane;
        const f32x2 ml = s < S ? *(const f32x2*)(sp.ml + 2 * (rowi * S + s)) : f32x2{-INFINITY, 0.f};
        mm[j] = ml[0]; ll[j] = ml[1];
        m = fmaxf(m, ml[0]);
    }
#pragma unroll
    for (int x = 32; x > 0; x >>= 1) m = fmaxf(m, __shfl_xor(m, x));
#pragma unroll
    for (int j = 0; j < NM; ++j) {
        w[j] = mm[j] == -INFINITY ? 0.f : exp2_hw((mm[j] - m) * p.scale_log2);
        l += ll[j] * w[j];
    }
#pragma unroll
    for (int x = 32; x > 0; x >>= 1) l += __shfl_xor(l, x);
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    static_assert(NL * NS == 64 || NL * NS == 128, "a batch of loads covers whole weight registers");
#pragma unroll
    for (int j = 0; j < kMaxSplits / (NL * NS); ++j) {
        if (j * NL * NS < S) {
            if (j > 0) load(j * NL * NS);
#pragma unroll
            for (int n = 0; n < NL; ++n) {
                constexpr int per = 64 / NS;                                  // splits of this batch per weight register
                const float ws = __shfl(w[j * NL / per + n / per], (sl + n * NS) & 63);   // 0 past S
                acc += v[n] * ws;
            }
        }
    }
    *(f32x4*)&red[sl][d] = acc;
    __syncthreads();
    if (tid < D / 2) {
        float a0 = 0.f, a1 = 0.f;
#pragma unroll
        for (int n = 0; n < NS; ++n) { a0 += red[n][2 * tid]; a1 += red[n][2 * tid + 1]; }
        const float inv = l > 0.f ? 1.0f / l : 0.f;
        const int i = (int)(rowi % p.Sq);
        const size_t bh = rowi / p.Sq;
        const int hq = (int)(bh % p.Hq), b = (int)(bh / p.Hq);
        *(unsigned*)(p.o + b * p.o_sb + hq * p.o_sh + (long long)i * p.o_ss + 2 * tid) = pack_bf16x2(a0 * inv, a1 * inv);
        if (tid == 0 && p.lse != nullptr) p.lse[rowi] = l > 0.f ? m * p.scale + logf(l) : -INFINITY;
    }
}

template <int D, bool CAUSAL>
void launch_split(const AttnParams& p, const AttnSplit& sp, unsigned blocks, hipStream_t stream) {
    const dim3 grid(blocks), block(sp.waves * 64);
    if (sp.rb == 1 && sp.waves == 2) hipLaunchKernelGGL((attn_fwd_split<D, CAUSAL, 1, 2>), grid, block, 0, stream, p, sp);
    else if (sp.rb == 1) hipLaunchKernelGGL((attn_fwd_split<D, CAUSAL, 1, 4>), grid, block, 0, stream, p, sp);
    else if (sp.rb == 2) hipLaunchKernelGGL((attn_fwd_split<D, CAUSAL, 2, 4>), grid, block, 0, stream, p, sp);
    else hipLaunchKernelGGL((attn_fwd_split<D, CAUSAL, 4, 4>), grid, block, 0, stream, p, sp);
}

}  // namespace

// Up to 64 query positions (more fill the tiled kernel's workgroups) against more than 128 keys: with fewer there is
// nothing to cut, and the 128-row kernel's shorter start and end win (B128 Hq16 Hkv16 Sq1 Sk64 D128: 19 against 23 us,
// Sk128 28 against 33, Sk256 47 against 45; B2 Hq12 Hkv4 Sq20 Sk128 D64: 5.6 against 6.3, Sk256 7.6 both).
bool attn_split_sizes(int Sq, int Sk) { return Sq <= 64 && Sk > 128; }

bool attn_split_fits(const AttnParams& p) {
    const long long kv_ss = p.k_ss > p.v_ss ? p.k_ss : p.v_ss;
    return ((long long)p.Sk + 64) * kv_ss * 2 < (1LL << 32);      // byte offsets inside a head in 32 bits
}

// More than 64 query positions: only where the tiled kernel's 128-row workgroups leave most CUs without one (up to 160 of
// them on 256 CUs) and its time, 1.0 us (D 128) or 0.73 us (D 64) per 64 keys and 2 us, is clearly more than the cut's.
// Measured, tiled -> cut, B Hq Hkv Sq Sk D causal: 1 1 1 2048 18000 128: 268 -> 43 us; 1 32 8 128 8192 128: 126 -> 42;
// 1 8 1 1024 9000 128: 138 -> 61; 2 32 8 128 5000 128: 80 -> 42; 1 16 16 512 2500 128: 46 -> 29; 4 16 2 256 9000 128 (128
// workgroups): 139 -> 102; 2 16 16 512 8000 64 (128): 89 -> 63.  With 256 of them the tiled kernel's larger tiles win:
// 2 32 8 512 5000 128: 89 against 108; 8 32 8 100 2000 128: 40 against 55.
bool attn_split_pays(int B, int Hq, int Hkv, int Sq, int Sk, int D) {
    if (attn_split_sizes(Sq, Sk)) return true;
    if (Sq <= 64 || Sk < 512 || (long long)B * Hq * ((Sq + 127) / 128) > 160) return false;
    const AttnSplit sp = attn_split_plan(B, Hq, Hkv, Sq, Sk, D, 0);
    return sp.splits > 1 && sp.cost < 0.85 * (2.0 + (Sk + 63) / 64 * (D == 128 ? 1.0 : 0.73));
}

// Up to 64 query positions: whether this cut, or this kernel uncut, beats a 128-row workgroup per query head.  It does up to 64
// packed rows per kv head, and with more query heads than the chip holds workgroups at two per CU (or at D = 64 at one, where it
// is level with them).  Below, with four row blocks per workgroup, the 128-row kernel walks 64 keys in 1.45 us (D 128; 1.12 at
// D 64) with one workgroup per CU and 2.25 with two, this one 32 in 1.0 (0.75).  Measured, 128-row kernel against this one,
// B Hq Hkv Sq Sk D: uncut 1 8 1 32 6000 128: 131 / 174 us; 5 16 2 50 296 64: 9.2 / 10.7; 25 8 2 20 238 128: 9.3 / 11.8;
// 10 32 2 18 7419 128 (320 heads): 256 / 210; 45 8 1 17 967 128 (360): 39 / 34; cut 2 32 2 53 339 128: 11.9 / 15.1;
// 7 32 2 13 834 128: 24.8 / 17.1.  Estimates that are level within 3 % stay uncut, which takes no memory.
bool attn_split_wins(const AttnSplit& sp, int B, int Hq, int Sk, int D) {
    const long long heads = (long long)B * Hq;
    if (sp.rb < 4 || heads > (D == 128 ? 512 : 256)) return true;
    const int tiles = (Sk + 63) / 64;
    const double rows128 = D == 128 ? 3.7 + tiles * (heads <= 256 ? 1.45 : 2.25) : 2.9 + tiles * 1.12;
    return sp.cost < (sp.splits > 1 ? 0.97 : 1.0) * rows128;
}

// The cut with the least estimated time, in microseconds.  Measured: a step of a workgroup (one tile per key group;
// 64 KB per CU at RB = 1) takes 1.3 us while HBM is no limit, which 128 CUs reach together, and 2.7 us with all CUs at
// it; two workgroups of two wavefronts per CU hide each other's start and end, which pays from several rounds of them
// on; with two row blocks sharing tiles 0.9 and 2.2 us, with four 1.0 with one workgroup per CU and 1.25 with two (D 128; a
// third adds nothing) or 0.75 with up to two and 1.5 with four (D 64); the combine costs 4 us, its traffic and its workgroups.
// Estimate against measurement at D = 128, B Hq Hkv Sq Sk: 32 32 8 1 4096: 88 / 100 us (one split); 16 32 8 1 1000:
// 12 / 15 us (two splits: 16 / 18); 40 8 8 1 5000: 163 / 159 us with one split, 146 / 143 us with four.
AttnSplit attn_split_plan(int B, int Hq, int Hkv, int Sq, int Sk, int D, int splits) {
    AttnSplit best;
    const long long R = (long long)(Hq / Hkv) * Sq;
    best.rb = R <= 32 ? 1 : R <= 64 ? 2 : 4;
    best.row_wgs = (int)((R + 32 * best.rb - 1) / (32 * best.rb));
    best.part = nullptr; best.ml = nullptr;
    best.splits = 1; best.waves = 4;
    const long long base = (long long)B * Hkv * best.row_wgs;
    const int tiles = (Sk + kTileKeys - 1) / kTileKeys;
    const double rows = (double)B * Hq * Sq;
    double least = 1e300;
    for (int waves = 4; waves >= (best.rb == 1 ? 2 : 4); waves -= 2) {
        const int groups = waves / best.rb;
        const long long slots = best.rb == 1 ? (D == 128 ? 1024 : 2048) / waves : best.rb == 4 && D == 64 ? 1024 : 512;
        const double start = best.rb == 4 ? (D == 128 ? 5.0 : 3.0) : waves == 2 ? 0.5 : 1.5;
        const double full = best.rb == 1 ? 2.7 : best.rb == 2 ? 2.2 : D == 128 ? 1.25 : 1.5;
        const double alone = best.rb == 4 ? (D == 128 ? 1.0 : 0.75) : best.rb == 2 ? 0.9 : waves == 2 ? 2.0 : 1.3;
        const int most = (tiles + groups - 1) / groups;           // at least one tile per key group, unless the caller asks for more parts
        for (int s = splits ? splits : 1; s <= (splits ? splits : kMaxSplits) && (splits || s == 1 || s <= most); s += s < 16 ? 1 : s >> 3) {
            const double steps = (double)((tiles + (long long)s * groups - 1) / ((long long)s * groups));
            long long rest = base * s % slots;
            if (best.rb == 4) rest = (rest + 255) / 256 * 256;        // the CUs with one workgroup more set the time
            const double rounds = (double)(base * s / slots), part = (double)rest / (double)slots;
            const double step = full * part > alone ? full * part : alone;
            const double cost = (waves == 2 ? 1.5 : 0.0) + rounds * (start + steps * full) + (part > 0 ? start + steps * step : 0.0)
                              + (s > 1 ? 4.0 + rows * (s <= kFewSplits ? 0.0002 : 0.0013) + rows * s * (D + 2) * 1e-6 : 0.0);
            if (cost < least) { least = cost; best.splits = s; best.waves = waves; best.cost = cost; }
        }
    }
    return best;
}

size_t attn_split_bytes(int B, int Hq, int Sq, int D, int splits) {
    return splits <= 1 ? 0 : (size_t)B * Hq * Sq * splits * (D + 2) * sizeof(float);
}

int attn_split_launch(AttnParams p, int D, int causal, AttnSplit sp, void* workspace, hipStream_t stream) {
    const size_t rows = (size_t)p.B * p.Hq * p.Sq;
    const long long blocks = (long long)p.B * p.Hkv * sp.row_wgs * sp.splits;
    if (blocks >= (1LL << 31) || (sp.splits > 1 && rows >= (1ULL << 31))) return -2;
    if (sp.splits > 1) {
        sp.part = (float*)workspace;
        sp.ml = sp.part + rows * sp.splits * D;
    }
    if (D == 128) { if (causal) launch_split<128, true>(p, sp, (unsigned)blocks, stream); else launch_split<128, false>(p, sp, (unsigned)blocks, stream); }
    else          { if (causal) launch_split<64, true>(p, sp, (unsigned)blocks, stream);  else launch_split<64, false>(p, sp, (unsigned)blocks, stream); }
    if (hipGetLastError() != hipSuccess) return -1;
    if (sp.splits > 1) {
        if (sp.splits <= kFewSplits) {
            const unsigned per = 1024u / D, grid = ((unsigned)rows + per - 1) / per;
            if (D == 128) hipLaunchKernelGGL(attn_split_combine_few<128>, dim3(grid), dim3(256), 0, stream, p, sp, (unsigned)rows);
            else hipLaunchKernelGGL(attn_split_combine_few<64>, dim3(grid), dim3(256), 0, stream, p, sp, (unsigned)rows);
        } else if (D == 128) hipLaunchKernelGGL(attn_split_combine<128>, dim3((unsigned)rows), dim3(256), 0, stream, p, sp);
        else hipLaunchKernelGGL(attn_split_combine<64>, dim3((unsigned)rows), dim3(256), 0, stream, p, sp);
        if (hipGetLastError() != hipSuccess) return -1;
    }
    return 0;
}
