// Two 3x3 convolutions of a 32-channel bf16 net in one launch:
//   RES:   out = bf16(bf16(conv2(m)) + x),  m = relu(conv1(x))   (a residual block)
//   !RES:  out = relu(conv2(m)),            m = relu(conv1(x))   (two layers of the plain topology)
// The same MFMAs in the same order as two launches of k_conv_mfma<32, ...>, so the same bits; the
// intermediate tensor m exists in LDS only.
//
// Why: with 32 channels a conv is bound by memory (144 flop per byte, 96 with a skip), and a block of two
// convs moved x, m, m, x, out.  Here it moves x and out; the halo of 2 and the second reading of x come from L2 for the
// most part (on 113 bins of 96 x 96 71 MiB are fetched for 64 MiB of x).
//
// Tile: 16 x 32 outputs = 18 x 34 values of m = 20 x 36 pixels of x, a workgroup of 4 waves, two
// workgroups per CU (so that one's loads, barriers and stores run under the other's MFMAs).
// LDS (80 KB): conv1's weights (18 KB) + one buffer that holds the x patch, then m, then the staged output:
// conv1's results wait in accumulators until every wave has read the patch.  Pixels are 80 bytes apart:
// 16-byte reads of neighbouring pixels fall into distinct banks and a tap is a constant
// offset (an immediate of the read), which an XOR swizzle would not be.
// conv1: m is numbered linearly (612 values in 20 N-tiles of 32, 5 per wave; the row pitch of 34 is not a
// multiple of an N-tile and padding it to 64 columns would double the work): per k-step one weight
// and 5 activation fragments feed 5 MFMAs.
// conv2: a wave owns 4 rows of 32 pixels; its weights stay in registers for the whole launch, but for the few
// that LDS has room for, and an activation fragment feeds the up to 3 rows it belongs to: 6 reads per
// 12 MFMAs.  x's values for the residual add and the next tile's patch are requested before these MFMAs.
// Measured, residual net of 8 blocks on 121 bins of 96 x 96: 52-55 us per block against 35.3 + 43.3 us for the two
// launches, 64 tiles: 10.6 us.  113 bins with stores through the L2: 47-50 us (0.87-0.92 PFLOP/s executed, 11 % of it the halo of m), clock
// 1.88 GHz, matrix pipe busy 46 % and LDS 52 % of the CU's cycles, 2.9 TB/s; a row-wise conv1 that reads 22 % less LDS changed nothing.  None of
// them is the limit by itself: a whole call of 8 blocks on these bins, 410 us, takes 354 without the blocks' stores, 405 without the
// patches' loads, 406 without x's second reading, 328 without any of the three, 330 without conv1's products and 363 without conv2's.
#include "conv_mfma_common.h"

#define BTH 16
#define BTW 32
#define XPW (BTW + 4)
#define XPH (BTH + 4)
#define MPW (BTW + 2)
#define MPH (BTH + 2)
#define PIX 80                              // bytes between pixels in LDS (64 of them used)
#define W1_BYTES (18 * 1024)
#define W2_LDS 5                            // conv2's first fragments, in LDS
#define BLK_LDS (W1_BYTES + XPW * XPH * PIX + 256 + W2_LDS * 1024)     // + 64 biases; two workgroups fill a CU's 160 KB

static_assert(20 * 32 * PIX <= XPW * XPH * PIX, "m and the values past its end fit the buffer");
__device__ __forceinline__ uint32_t row34(uint32_t q) { return __umul24(q, 1928u) >> 16; }      // q / MPW for q < 640

struct block_args {
    const __bf16* in;         // [N][H][W][32]
    const uint4 *w1, *w2;     // fragment order, [tap][k-step][lane][8]
    const float *b1, *b2;
    __bf16* out;              // not `in`: neighbouring tiles read its halo
    const uint32_t* n_valid;
    int N, H, W, rev;
};

template <bool RES>
__global__ __launch_bounds__(256, 2) void k_block32(block_args a)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint8_t* buf = lds + W1_BYTES;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lx = lane & 31, hi = lane >> 5;
    const int n_img = a.n_valid ? min((int)*a.n_valid, a.N) : a.N;
    const int tiles_x = (a.W + BTW - 1) / BTW, tiles_y = (a.H + BTH - 1) / BTH, tiles_img = tiles_x * tiles_y;
    const int n_tiles = n_img * tiles_img, G = gridDim.x;
    // whole rounds: neighbouring tiles on one XCD (workgroups are dealt round-robin to the 8 XCDs);
    // the last, partial round in launch order, which spreads it over all XCDs and CUs
    const int wg = (G % 8 == 0) ? (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8 : blockIdx.x;
    auto tile_of = [&](int round) __attribute__((always_inline)) {
        const int t = round * G + ((round + 1) * G <= n_tiles ? wg : (int)blockIdx.x);
        return t >= n_tiles ? -1 : (a.rev ? n_tiles - 1 - t : t);
    };
    const uint32_t img_bytes = (uint32_t)a.H * a.W * 64;

    constexpr int NP = (XPW * XPH * 4 + 255) / 256;          // 16-byte pieces of the patch per thread
    uint4 pre[NP];
    auto load_patch = [&](int tile) __attribute__((always_inline)) {
        const int n = tile / tiles_img, tr = tile - n * tiles_img, ty = tr / tiles_x, y0 = ty * BTH, x0 = (tr - ty * tiles_x) * BTW;
        __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc((void*)(a.in + (size_t)n * a.H * a.W * 32), 0, img_bytes, RSRC_FLAGS);
        uint32_t t = tid;
        asm volatile("" : "+v"(t));                          // keeps the pieces' coordinates out of the loop's registers
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const uint32_t idx = t + 256 * j, row = __umul24(idx, 58255u) >> 23, px = (idx - __umul24(row, XPW * 4)) >> 2;      // idx / 144 for idx < 4096
            const int gx = x0 - 2 + (int)px;                 // a row outside the image is an offset outside the descriptor's range
            const uint32_t off = (uint32_t)(__mul24(y0 - 2 + (int)row, a.W) + gx) * 64u + (idx & 3) * 16;
            const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rin, (uint32_t)gx < (uint32_t)a.W ? off : OOB_OFF, 0, 0);
            pre[j] = make_uint4(v[0], v[1], v[2], v[3]);
        }
    };

    int round = 0, tile = tile_of(0);
    if (tile < 0) return;                                    // the whole workgroup
    load_patch(tile);
    for (int i = tid; i < W1_BYTES / 16; i += 256) ((uint4*)lds)[i] = a.w1[i];
    bf16x8 w2[18];                                           // [(kx * 2 + k-step) * 3 + ky]; the first W2_LDS are not kept in registers
    uint8_t* w2l = buf + XPW * XPH * PIX + 256;
#pragma unroll
    for (int k = 0; k < 18; ++k) {
        const uint4* src = a.w2 + (((k % 3) * 3 + k / 6) * 2 + k / 3 % 2) * 64 + lane;
        if (k >= W2_LDS) w2[k] = *(const bf16x8*)src;
        else if ((k & 3) == wave) *(uint4*)(w2l + k * 1024 + lane * 16) = *src;
    }
    // biases in LDS (in registers they would take 32); in accumulator layout a lane holds channels 8*(e/4) + 4*hi + e%4
    float* bias = (float*)(buf + XPW * XPH * PIX);
    if (tid < 64) bias[tid] = tid < 32 ? a.b1[tid] : a.b2[tid - 32];
    const uint8_t* blane = (const uint8_t*)bias + hi * 16;

    const uint32_t p_dst = (tid >> 2) * PIX + (tid & 3) * 16;
    while (tile >= 0) {
        const int n = tile / tiles_img, tr = tile - n * tiles_img, ty = tr / tiles_x, y0 = ty * BTH, x0 = (tr - ty * tiles_x) * BTW;
        lds_barrier();                                       // the previous tile's staged values are read
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            if (j < NP - 1 || tid < XPW * XPH * 4 - 256 * (NP - 1)) *(uint4*)(buf + p_dst + j * 64 * PIX) = pre[j];
        }
        lds_barrier();                                       // patch and weights visible
        {
            // N-tile j of the wave covers m[(wave*5 + j)*32 ..]; values past the last one repeat it and are dropped
            int q0 = wave * 160 + lx;
            asm volatile("" : "+v"(q0));                     // not kept over the tiles (registers)
            uint32_t m_src[5];
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                const uint32_t q = min(q0 + j * 32, MPW * MPH - 1);
                m_src[j] = __umul24(q + row34(q) * (XPW - MPW), PIX) + hi * 16;
            }
            f32x16 acc[5];
            f32x16 bv;                                       // the first MFMA's C operand
#pragma unroll
            for (int q = 0; q < 4; ++q) { const float4 b = *(const float4*)(blane + q * 32); bv[4 * q] = b.x; bv[4 * q + 1] = b.y; bv[4 * q + 2] = b.z; bv[4 * q + 3] = b.w; }
            bf16x8 A[2], B[2][5];
            auto frag = [&](int k, int s) __attribute__((always_inline)) {
                const int st = k / 3, ky = k % 3, kx = st >> 1, ks = st & 1;
                A[s] = *(const bf16x8*)(lds + ((((ky * 3 + kx) * 2 + ks) << 10) + lane * 16));
#pragma unroll
                for (int j = 0; j < 5; ++j) B[s][j] = *(const bf16x8*)(buf + m_src[j] + ((ky * XPW + kx) * PIX + ks * 32));
            };
            frag(0, 0);
#pragma unroll
            for (int k = 0; k < 18; ++k) {
                if (k < 17) frag(k + 1, (k + 1) & 1);
#pragma unroll
                for (int j = 0; j < 5; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[k & 1], B[k & 1][j], k ? acc[j] : bv, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            lds_barrier();                                   // the patch is read by every wave: m takes its place
            asm volatile("" : "+v"(q0));
#pragma unroll
            for (int j = 0; j < 5; ++j) {
                const uint32_t p = q0 + j * 32, y = row34(p), gy = y0 - 1 + y, gx = x0 - 1 + (p - __umul24(y, MPW));
                const uint32_t in = (gy < (uint32_t)a.H & gx < (uint32_t)a.W) ? ~0u : 0u;      // conv2's zero padding
                uint8_t* dst = buf + __umul24(p, PIX) + hi * 8;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    uint2 pk;
                    pk.x = relu_bf16x2(pack_bf16x2(acc[j][4 * q], acc[j][4 * q + 1])) & in;
                    pk.y = relu_bf16x2(pack_bf16x2(acc[j][4 * q + 2], acc[j][4 * q + 3])) & in;
                    *(uint2*)(dst + q * 16) = pk;
                }
            }
        }
        lds_barrier();                                       // m visible
        const int next = tile_of(++round);
        __amdgpu_buffer_rsrc_t rsk = __builtin_amdgcn_make_buffer_rsrc((void*)(a.in + (size_t)n * a.H * a.W * 32), 0, RES ? img_bytes : 0u, RSRC_FLAGS);
        __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc((void*)(a.out + (size_t)n * a.H * a.W * 32), 0, img_bytes, RSRC_FLAGS);
        auto out_off = [&](int j, int l) __attribute__((always_inline)) {        // output piece j of lane l
            const int y = y0 + wave * 4 + (j >> 1), x = x0 + (j & 1) * 16 + (l >> 2);
            return x < a.W ? (uint32_t)(__mul24(y, a.W) + x) * 64u + (l & 3) * 16 : OOB_OFF;
        };
        f32x16 acc[4];
        uint4 sk[RES ? 8 : 1];
        {
            f32x16 bv;
#pragma unroll
            for (int q = 0; q < 4; ++q) { const float4 b = *(const float4*)(blane + 128 + q * 32); bv[4 * q] = b.x; bv[4 * q + 1] = b.y; bv[4 * q + 2] = b.z; bv[4 * q + 3] = b.w; }
            if constexpr (RES) {
                int l = lane;
                asm volatile("" : "+v"(l));
#pragma unroll
                for (int j = 0; j < 8; ++j) {                // x again, from L2
                    const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsk, out_off(j, l), 0, 0);
                    sk[j] = make_uint4(v[0], v[1], v[2], v[3]);
                }
            }
            if (next >= 0) load_patch(next);
            const uint8_t* mrow = buf + (wave * 4 * MPW + lx) * PIX + hi * 16;
#pragma unroll
            for (int st = 0; st < 6; ++st) {
                bf16x8 B[6];
#pragma unroll
                for (int ky = 0; ky < 3; ++ky)
                    if (st * 3 + ky < W2_LDS) w2[st * 3 + ky] = *(const bf16x8*)(w2l + (st * 3 + ky) * 1024 + lane * 16);
#pragma unroll
                for (int py = 0; py < 6; ++py) B[py] = *(const bf16x8*)(mrow + (py * MPW + (st >> 1)) * PIX + (st & 1) * 32);
#pragma unroll
                for (int py = 0; py < 6; ++py)
#pragma unroll
                    for (int ky = 0; ky < 3; ++ky)
                        if (py - ky >= 0 && py - ky < 4) acc[py - ky] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w2[st * 3 + ky], B[py], st + ky ? acc[py - ky] : bv, 0, 0, 0);
            }
        }
        lds_barrier();                                       // m is read by every wave
        uint8_t* stg = buf + wave * (4 * 32 * PIX);          // the wave's own slice
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint2 pk;
                pk.x = pack_bf16x2(acc[r][4 * q], acc[r][4 * q + 1]); pk.y = pack_bf16x2(acc[r][4 * q + 2], acc[r][4 * q + 3]);
                if constexpr (!RES) { pk.x = relu_bf16x2(pk.x); pk.y = relu_bf16x2(pk.y); }
                *(uint2*)(stg + (r * 32 + lx) * PIX + q * 16 + hi * 8) = pk;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        int l = lane;
        asm volatile("" : "+v"(l));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            uint4 o = *(const uint4*)(stg + (j * 16 + (l >> 2)) * PIX + (l & 3) * 16);
            if constexpr (RES) {
                o.x = pack_bf16x2(bf16_lo(o.x) + bf16_lo(sk[j].x), bf16_hi(o.x) + bf16_hi(sk[j].x));
                o.y = pack_bf16x2(bf16_lo(o.y) + bf16_lo(sk[j].y), bf16_hi(o.y) + bf16_hi(sk[j].y));
                o.z = pack_bf16x2(bf16_lo(o.z) + bf16_lo(sk[j].z), bf16_hi(o.z) + bf16_hi(sk[j].z));
                o.w = pack_bf16x2(bf16_lo(o.w) + bf16_lo(sk[j].w), bf16_hi(o.w) + bf16_hi(sk[j].w));
            }
            const i32x4 v = {(int)o.x, (int)o.y, (int)o.z, (int)o.w};
            __builtin_amdgcn_raw_buffer_store_b128(v, rout, out_off(j, l), 0, ST_THROUGH);
        }
        tile = next;
    }
}

template <bool RES>
static hipError_t launch(hipStream_t stream, int device, int n_cu, const block_args& a)
{
    static bool attr_done[RH_MAX_DEVICES] = {};              // the attribute is per device
    if (!attr_done[device]) {
        hipError_t e = hipFuncSetAttribute((const void*)k_block32<RES>, hipFuncAttributeMaxDynamicSharedMemorySize, BLK_LDS);
        if (e != hipSuccess) return e;
        attr_done[device] = true;
    }
    hipLaunchKernelGGL((k_block32<RES>), dim3(2 * n_cu), dim3(256), BLK_LDS, stream, a);
    return hipSuccess;
}

hipError_t rh_launch_block32(rh_ctx* ctx, const rh_layer& L1, const rh_layer& L2, const __bf16* in, __bf16* out, int N, int H, int W,
                             bool res, const uint32_t* n_valid)
{
    block_args a;
    const uint8_t* wp = (const uint8_t*)ctx->wpack;
    a.in = in; a.out = out; a.n_valid = n_valid; a.N = N; a.H = H; a.W = W;
    a.w1 = (const uint4*)(wp + L1.wp_off); a.w2 = (const uint4*)(wp + L2.wp_off);
    a.b1 = ctx->bpack + L1.bp_off; a.b2 = ctx->bpack + L2.bp_off;
    a.rev = (ctx->conv_parity ^= 1);                         // start on what the previous launch touched last
    return res ? launch<true>(ctx->stream, ctx->device, ctx->n_cu, a) : launch<false>(ctx->stream, ctx->device, ctx->n_cu, a);
}
