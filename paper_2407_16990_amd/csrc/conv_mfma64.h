// The products of one unit of the 64-channel body convs - 8 x 32 pixels, 64 input and 64 output channels - as a wave of the two-team
// kernels (conv_mfma_duo.hip, conv_body.hip) does them: 2 rows of 32 pixels, all output channels, both operands in LDS.
//
// v_mfma_f32_16x16x32_bf16, D[cout][pixel]: 16 tiles of 16 channels x 16 pixels, 64 accumulator registers.  Half the size of a 32x32x16
// product, at the same rate and with the same fragments (1 KB of A and B for a wave's 64 x 64 block and 32 of K either way), but it
// takes less power, and the chip is at its limit here: from registers, operands N(0, 1), 1.73 PFLOP/s with 32x32x16 and 1.90 to 2.03 with this,
// the more the fewer operands change from one product to the next.  With 32x32x16 / this, us: EDSR x4 on 76 bins of 128 x 128 3 031 / 2 944, 150 bins
// 5 972 / 5 800, 16 whole frames of 480 x 272 5 050 / 4 950; a chain of single half tiles (conv_body.hip, 3 bins) 311 / 315.
#pragma once
#include <type_traits>

#include "conv_mfma_common.h"

#define PW 34                            // patch columns: 32 and the two beside them
#define C64_SUBSTEPS 18                  // (ky, kx, half of K), 16 products each

struct conv64_acc { f32x4 v[2][2][4]; };                     // [row][half of its pixels][16 channels]

// Lane l holds channels 16 m + 4 (l / 16) + {0..3} of pixel l % 16 of each tile.
__device__ __forceinline__ void conv64_bias(f32x4 (&b)[4], const float* bias, int lane)
{
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const float4 v = *(const float4*)(bias + m * 16 + (lane >> 4) * 4);
        b[m][0] = v.x; b[m][1] = v.y; b[m][2] = v.z; b[m][3] = v.w;
    }
}

template <int N, int I = 0, typename F>
__device__ __forceinline__ void conv64_each(F& f)
{
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); conv64_each<N, I + 1>(f); }
}

// wlane: the weights in LDS, [tap][half of K][m][lane][8], + 16 lane.  prow: the patch row above the wave's first, 16-byte channel
// groups of a pixel swizzled by its column.  The sums start from the bias, as the first products' C operand, and run over
// (ky, kx, half of K) in this order in every kernel of the body, so that all give the same bits.
// The fragments of a sub-step are read during the one before, into the other of two register sets.  hook(sub-step): what the kernel
// does between two sub-steps.
template <typename H>
__device__ __forceinline__ void conv64_products(conv64_acc& acc, const f32x4 (&bias)[4], const uint8_t* wlane, const uint8_t* prow, int lane, H& hook)
{
    bf16x8 A[2][4], B[2][2][2];
    const int px0 = lane & 15, grp = lane >> 4;
    auto load = [&](int st, int i) __attribute__((always_inline)) {        // fragment i of 8 of sub-step st
        const int ky = st / 6, kx = st / 2 % 3, kh = st & 1, set = st & 1;
        if (i >= 2 && i < 6) { A[set][i - 2] = *(const bf16x8*)(wlane + ((((ky * 3 + kx) * 2 + kh) * 4 + i - 2) << 10)); return; }
        const int px = px0 + kx, r = i >> 2, n = i & 1;
        B[set][r][n] = *(const bf16x8*)(prow + px * 128 + (((grp ^ (px & 7)) << 4) ^ (kh << 6)) + (ky + r) * (PW * 128) + n * 2048);
    };
#pragma unroll
    for (int i = 0; i < 8; ++i) load(0, i);
    auto sub = [&](auto st_c) __attribute__((always_inline)) {
        constexpr int st = decltype(st_c)::value, set = st & 1;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            if (st + 1 < C64_SUBSTEPS && (k & 1) == 0) load(st + 1, k >> 1);
            const int r = k >> 3, m = k >> 1 & 3, n = k & 1;
            acc.v[r][n][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[set][m], B[set][r][n], st == 0 ? bias[m] : acc.v[r][n][m], 0, 0, 0);
            if (k & 1) __builtin_amdgcn_sched_barrier(0);
        }
        hook(st_c);
    };
    conv64_each<C64_SUBSTEPS>(sub);
}

// Four sums of a lane as bf16, and where these 8 bytes go in the wave's slice of 2 x 32 pixels of 128 bytes, swizzled by the pixel like a patch.
__device__ __forceinline__ uint2 conv64_round(const f32x4& v)
{
    uint2 pk;
    pk.x = pack_bf16x2(v[0], v[1]); pk.y = pack_bf16x2(v[2], v[3]);
    return pk;
}
__device__ __forceinline__ uint32_t conv64_slot(int r, int n, int m, int lane)
{
    return (uint32_t)((r * 32 + n * 16 + (lane & 15)) * 128 + (((m * 2 + (lane >> 5)) ^ (lane & 7)) << 4) + (lane >> 4 & 1) * 8);
}
