// bf16 GEMM for operands whose rows start at any 2-byte address (sizes, pitches or pointers that are no multiples of
// 16 bytes): MFMA tiles fed through registers.
//
// The direct HBM -> LDS copies of the aligned kernel want 16-byte aligned pieces; an ordinary vector load does not
// (global memory is in unaligned access mode on this target: a 16-byte load may start at any address and costs at most
// one more cache line).  So a 16-byte piece goes global -> registers -> the same XOR-swizzled LDS tiles the aligned
// kernel reads its operands from (gemm_layout.h), PF stages ahead in registers, two stages in LDS, one barrier per stage.
//
// No access leaves the operands, and no load is guarded inside the loop: rows past the last one re-read it, the last
// column tile of B stored [K,N] starts at N - BN, and the last stage starts at K - 64; what an overlapping stage has
// seen before is zeroed on its way to LDS in both operands (0 x inf would be NaN), and columns a neighbouring tile owns
// are not stored.  That needs K >= 64 and, for B stored [K,N], N >= BN.
//
// What bounds it: a workgroup has one wavefront per SIMD, which waits for its loads, writes LDS, meets the barrier and multiplies in
// turn.  M999 N2001 K1501 [K,N] on 64 x 64 tiles, two workgroups per CU, reads 786 KB per CU in 20.5 us; on 256 tiles of 128 x 64 it
// is 590 KB and 18.6 us, 32 bytes per ns and CU, where copies alone reach 60 to 118 from L2.  The fp32 FMA kernel that served these
// sizes needed 252 us.  M2001 N2001 K2001 on 128 x 128 tiles: 35.6 us (450 TFLOP/s).
#include <stdint.h>

#include "gemm_layout.h"
#include "gemm_launch.h"
#include "gfx950_prims.h"

namespace {

using namespace gemm_layout;
using namespace gfx950;

typedef __attribute__((ext_vector_type(4), aligned(2))) unsigned u32x4_any;      // 16 bytes at any 2-byte address

constexpr int kUBK = 64;                         // reduction depth of a stage: 128-byte rows of A and of B stored [N,K]

// BM x BN tile, WM x WN wavefronts of (BM / WM) x (BN / WN), PF stages in registers.
template <int BM_, int BN_, int WM_, int WN_, int PF_> struct UTile {
    static constexpr int BM = BM_, BN = BN_, WM = WM_, WN = WN_, PF = PF_;
    static constexpr int kThreads = WM * WN * 64;
    static constexpr int kMB = BM / WM / 32, kNB = BN / WN / 32;
    static constexpr int kStageA = BM * 128, kStageB = BN * 128, kStage = kStageA + kStageB;
    static constexpr int kPA = BM * 8 / kThreads, kPB = BN * 8 / kThreads;      // 16-byte pieces per thread and stage
    static constexpr int kCPitch = BN * 2 + 16;                                  // bytes per row of the staged result
    static constexpr int kLds = 2 * kStage > BM * kCPitch ? 2 * kStage : BM * kCPitch;
    static_assert(kMB >= 1 && kNB >= 1 && kPA >= 1 && kPB >= 1 && (PF == 2 || PF == 4), "unsupported tile");
};
using USmall = UTile<64, 64, 2, 2, 4>;
using UTall = UTile<128, 64, 2, 2, 4>;
using ULarge = UTile<128, 128, 2, 2, 2>;

// keep elements e >= z of the eight starting at element `first`
__device__ __forceinline__ u32x4 keep_from(u32x4 v, int first, int z) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const int e = first + 2 * d;
        const unsigned mask = (e >= z ? 0x0000ffffu : 0u) | (e + 1 >= z ? 0xffff0000u : 0u);
        v[d] &= mask;
    }
    return v;
}

template <class T, bool B_NK>
__global__ __launch_bounds__(T::kThreads) void gemm_bf16_unaligned(GemmParams p) {
    constexpr int BM = T::BM, BN = T::BN, PF = T::PF, PA = T::kPA, PB = T::kPB, RB = 2 * BN;
    __shared__ __attribute__((aligned(16))) char smem[T::kLds];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % T::WM, wn = wave / T::WM;
    const int M = p.M, N = p.N, K = p.K;
    const TileCoord tc = tile_coord(blockIdx.x, gridDim.x, p.tiles_m, p.tiles_n);
    const int m0 = tc.tm * BM;
    const int n_own = tc.tn * BN;                               // columns from here on are this tile's
    const int n0 = B_NK ? n_own : min(n_own, N - BN);           // first column it computes
    const int nK = (K + kUBK - 1) / kUBK;
    const int z = nK * kUBK - K;                                // elements the last stage shares with the one before

    // piece t of this thread: row and 16-byte chunk of the tile
    const __bf16* a_src[PA];
    const __bf16* b_src[PB];
    int a_dst[PA], b_dst[PB];
#pragma unroll
    for (int t = 0; t < PA; ++t) {
        const int i = tid + t * T::kThreads, row = i >> 3, chunk = i & 7;
        a_src[t] = p.a + (long long)min(m0 + row, M - 1) * p.lda + 8 * chunk;
        a_dst[t] = kt_offset(row, chunk);
    }
#pragma unroll
    for (int t = 0; t < PB; ++t) {
        const int i = tid + t * T::kThreads;
        if constexpr (B_NK) {
            const int row = i >> 3, chunk = i & 7;
            b_src[t] = p.b + (long long)min(n0 + row, N - 1) * p.ldb + 8 * chunk;
            b_dst[t] = T::kStageA + kt_offset(row, chunk);
        } else {
            const int krow = i / (BN / 8), chunk = i % (BN / 8);
            b_src[t] = p.b + (long long)krow * p.ldb + n0 + 8 * chunk;
            b_dst[t] = T::kStageA + nt_offset<RB>(krow, chunk);
        }
    }
    u32x4 ra[PF][PA], rb[PF][PB];
    auto fetch = [&](auto set, int U) __attribute__((always_inline)) {
        const int k0 = U >= nK - 1 ? K - kUBK : U * kUBK;          // (past the end: the last stage again, never used)
        const long long b_off = B_NK ? (long long)k0 : (long long)k0 * p.ldb;
#pragma unroll
        for (int t = 0; t < PA; ++t) ra[set.value][t] = *(const u32x4_any*)(a_src[t] + k0);
#pragma unroll
        for (int t = 0; t < PB; ++t) rb[set.value][t] = *(const u32x4_any*)(b_src[t] + b_off);
    };
    auto put = [&](auto set, int U, int buf) __attribute__((always_inline)) {
        if (U == nK - 1 && z > 0) {
#pragma unroll
            for (int t = 0; t < PA; ++t) ra[set.value][t] = keep_from(ra[set.value][t], 8 * ((tid + t * T::kThreads) & 7), z);
#pragma unroll
            for (int t = 0; t < PB; ++t) {
                const int i = tid + t * T::kThreads;
                if constexpr (B_NK) rb[set.value][t] = keep_from(rb[set.value][t], 8 * (i & 7), z);
                else if (i / (BN / 8) < z) rb[set.value][t] = u32x4{0u, 0u, 0u, 0u};
            }
        }
#pragma unroll
        for (int t = 0; t < PA; ++t) *(u32x4*)(smem + buf * T::kStage + a_dst[t]) = ra[set.value][t];
#pragma unroll
        for (int t = 0; t < PB; ++t) *(u32x4*)(smem + buf * T::kStage + b_dst[t]) = rb[set.value][t];
    };

    f32x16 acc[T::kNB][T::kMB];
#pragma unroll
    for (int in = 0; in < T::kNB; ++in)
#pragma unroll
        for (int jm = 0; jm < T::kMB; ++jm)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[in][jm][r] = 0.0f;

    auto compute = [&](int buf) __attribute__((always_inline)) {
        const char* const sA = smem + buf * T::kStage;
        const char* const sB = sA + T::kStageA;
#pragma unroll
        for (int ks = 0; ks < kUBK / 16; ++ks) {
            bf16x8 fa[T::kMB], fb[T::kNB];
#pragma unroll
            for (int jm = 0; jm < T::kMB; ++jm) fa[jm] = *(const bf16x8*)(sA + kt_offset(kt_row(wm * T::kMB + jm, lane), kt_chunk(ks, lane)));
#pragma unroll
            for (int in = 0; in < T::kNB; ++in) {
                if constexpr (B_NK) {
                    fb[in] = *(const bf16x8*)(sB + kt_offset(kt_row(wn * T::kNB + in, lane), kt_chunk(ks, lane)));
                } else {
                    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, sB + tr_offset<RB>(wn * T::kNB + in, ks, 0, lane)));
                    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(s16x4, sB + tr_offset<RB>(wn * T::kNB + in, ks, 1, lane)));
                    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    fb[in] = __builtin_bit_cast(bf16x8, v);
                }
            }
#pragma unroll
            for (int jm = 0; jm < T::kMB; ++jm)
#pragma unroll
                for (int in = 0; in < T::kNB; ++in) acc[in][jm] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[in], fa[jm], acc[in][jm], 0, 0, 0);
        }
    };
    // own LDS reads and writes done, then everybody's; loads into registers stay in flight
    auto sync_lds = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(0xC07F);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

    // stage U lives in register set U % PF from PF stages before its turn, and in LDS buffer U & 1.  The loads of the
    // main loop are not conditional, so that a wait covers exactly the stage it is for.
    static_for<0, PF>([&](auto s) __attribute__((always_inline)) { fetch(s, s.value); });
    put(IntC<0>{}, 0, 0);
    fetch(IntC<0>{}, PF);
    sync_lds();
    int U0 = 0;
    for (; U0 + PF <= nK; U0 += PF)
        static_for<0, PF>([&](auto s) __attribute__((always_inline)) {
            constexpr int nxt = (s.value + 1) % PF;
            compute(s.value & 1);
            put(IntC<nxt>{}, U0 + s.value + 1, (s.value + 1) & 1);      // (the barrier at the end of the stage before freed that buffer)
            fetch(IntC<nxt>{}, U0 + s.value + 1 + PF);
            sync_lds();
        });
    static_for<0, PF - 1>([&](auto s) __attribute__((always_inline)) {
        if (U0 + s.value < nK) {
            compute(s.value & 1);
            put(IntC<(s.value + 1) % PF>{}, U0 + s.value + 1, (s.value + 1) & 1);
            sync_lds();
        }
    });

    // result: lanes hold 4 consecutive n of one row m; through LDS so that rows leave in 16-byte pieces
    const int half = lane >> 5;
#pragma unroll
    for (int in = 0; in < T::kNB; ++in)
#pragma unroll
        for (int jm = 0; jm < T::kMB; ++jm)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int m = (wm * T::kMB + jm) * 32 + (lane & 31), n = (wn * T::kNB + in) * 32 + 8 * g + 4 * half;
                u32x2 v;
                v[0] = pack_bf16x2(acc[in][jm][4 * g + 0], acc[in][jm][4 * g + 1]);
                v[1] = pack_bf16x2(acc[in][jm][4 * g + 2], acc[in][jm][4 * g + 3]);
                *(u32x2*)(smem + m * T::kCPitch + 2 * n) = v;
            }
    sync_lds();
#pragma unroll
    for (int t = 0; t < BM * (BN / 8) / T::kThreads; ++t) {
        const int i = tid + t * T::kThreads, row = i / (BN / 8), col = 8 * (i % (BN / 8));
        if (m0 + row >= M) continue;
        const u32x4 v = *(const u32x4*)(smem + row * T::kCPitch + 2 * col);
        __bf16* const dst = p.c + (long long)(m0 + row) * p.ldc + n0 + col;
        if (n0 + col >= n_own && n0 + col + 8 <= N) {
            *(u32x4_any*)dst = v;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (n0 + col + e >= n_own && n0 + col + e < N) ((unsigned short*)dst)[e] = (unsigned short)(v[e >> 1] >> (16 * (e & 1)));
        }
    }
}

template <class T>
void launch_unaligned(GemmParams p, int b_is_nk, hipStream_t stream) {
    p.tiles_m = (p.M + T::BM - 1) / T::BM;
    p.tiles_n = (p.N + T::BN - 1) / T::BN;
    const dim3 grid((unsigned)(p.tiles_m * p.tiles_n)), block(T::kThreads);
    if (b_is_nk) hipLaunchKernelGGL((gemm_bf16_unaligned<T, true>), grid, block, 0, stream, p);
    else         hipLaunchKernelGGL((gemm_bf16_unaligned<T, false>), grid, block, 0, stream, p);
}

}  // namespace

// One whole stage along k, and one whole tile along n where the rows of B run along n.
bool gemm_unaligned_sizes(int N, int K, int b_is_nk) { return K >= kUBK && (b_is_nk || N >= USmall::BN); }

void gemm_unaligned_launch(const GemmParams& p, int b_is_nk, int tile, hipStream_t stream) {
    tile = unaligned_tile(p.M, p.N, b_is_nk != 0, tile);
    if (tile == 1284) launch_unaligned<UTall>(p, b_is_nk, stream);
    else if (tile == 128) launch_unaligned<ULarge>(p, b_is_nk, stream);
    else launch_unaligned<USmall>(p, b_is_nk, stream);
}
