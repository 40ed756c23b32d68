// SR forward, fp32 path (Sec. 3.3.3): direct 3x3 convolutions on the vector ALUs.
// This is the high-precision path (configurations whose weights and activations are fp32);
// the throughput path is the bf16 MFMA one in conv_mfma.hip.
#include <type_traits>

#include "rh_internal.h"

#define CO_T 8   // output channels per thread

// Thread = one pixel x CO_T output channels.  The output-channel block is uniform over the
// workgroup, so the weights are read through the scalar unit.  Input: f32 NHWC, or the u8
// image (then x/255 is taken here).  Epilogue: bias, optional ReLU, optional skip add,
// optional pixel shuffle by ps into out[N][H*ps][W*ps][Cout/ps^2].
__global__ __launch_bounds__(256) void k_conv3x3_f32(const void* __restrict__ in_, int in_u8,
                                                     const float* __restrict__ w, const float* __restrict__ bias,
                                                     float* out, const float* skip,
                                                     int H, int W, int Cin, int Cout, int relu, int ps,
                                                     const uint32_t* __restrict__ n_valid, int tiles_x)
{
    const int n = blockIdx.z;
    if (n_valid && (uint32_t)n >= *n_valid) return;
    const int tid = threadIdx.x, ty = blockIdx.x / tiles_x, tx = blockIdx.x - ty * tiles_x;
    const int x = tx * 16 + (tid & 15), y = ty * 16 + (tid >> 4);
    const int co0 = blockIdx.y * CO_T;
    if (x >= W || y >= H) return;
    float acc[CO_T];
    int cj[CO_T];
#pragma unroll
    for (int j = 0; j < CO_T; ++j) { cj[j] = min(co0 + j, Cout - 1); acc[j] = bias[cj[j]]; }
    const float* inf = (const float*)in_;
    const uint8_t* inb = (const uint8_t*)in_;
    for (int ky = 0; ky < 3; ++ky) {
        const int yy = y + ky - 1;
        if (yy < 0 || yy >= H) continue;
        for (int kx = 0; kx < 3; ++kx) {
            const int xx = x + kx - 1;
            if (xx < 0 || xx >= W) continue;
            const size_t pix = ((size_t)n * H + yy) * W + xx;
            const int tap = ky * 3 + kx;
            for (int ci = 0; ci < Cin; ++ci) {
                const float v = in_u8 ? __fdiv_rn((float)inb[pix * Cin + ci], 255.0f) : inf[pix * Cin + ci];
#pragma unroll
                for (int j = 0; j < CO_T; ++j) acc[j] = fmaf(w[((size_t)cj[j] * 9 + tap) * Cin + ci], v, acc[j]);
            }
        }
    }
    const int r2 = ps * ps, Co = Cout / r2;
#pragma unroll
    for (int j = 0; j < CO_T; ++j) {
        const int co = co0 + j;
        if (co >= Cout) break;
        float v = acc[j];
        if (relu) v = fmaxf(v, 0.0f);
        const int c = co / r2, sub = co - c * r2, si = sub / ps, sj = sub - si * ps;
        const size_t o = (((size_t)n * H * ps + (size_t)y * ps + si) * (W * ps) + (size_t)x * ps + sj) * Co + c;
        if (skip) v += skip[o];
        out[o] = v;
    }
}

// The same convolution for up to LDS_CIN input channels, from a patch in LDS: thread = one pixel x 4
// output channels, workgroup = 16 x 16 pixels.  The kernel above is bound by the latency of its
// loads: every input value of a lane comes from a line of its own (a pixel's channels are
// contiguous), nine times, with one wave per SIMD in flight on small batches.  Here the 18 x 18
// pixel patch is fetched once as contiguous 16-byte pieces, all of a thread's pieces in flight
// together, and read back four channels at a time (pixel pitch Cin + 4 floats); the weights are laid
// out [co / 4][tap][ci][4], so that the scalar unit fetches 16 of them with one load.  Same products
// in the same order: results are bit for bit those of the kernel above.
// Measured, whole networks: 8 bins of 64 x 64, 4 layers of 16 channels: 98.9 -> 34.5 us; residual net, 7
// layers of 32 channels, 4 x 96 x 96: 1455 -> 234; EDSR with 64 channels, 64 x 96 x 96: 86.9 -> 25.3 ms.
// The line lies where the patch stops fitting a CU's LDS (120 channels: 157 of 160 KB), because a single workgroup
// per CU still gains.  Kernel above -> patch, EDSR x4 of 2 blocks on 16 x 128 x 128: 68 channels 150 -> 52 ms,
// 96: 268 -> 100, 120: 436 -> 156; 4 plain layers on one image of 64 x 64: 377 -> 116, 529 -> 155, 663 -> 186 us.
#define CO_L 4
#define LDS_CIN 120
static_assert(18 * 18 * (LDS_CIN + 4) * sizeof(float) <= 160 * 1024, "the patch fits the LDS of a CU");

//
// CIN: the number of input channels where it is known (the first conv's 3, nets of 16 and 32 channels), or 0.  On a
// small batch a conv is a chain of latencies - the image count, the patch, a scalar load for every four channels and
// tap - around a microsecond of products: with CIN all of a thread's pieces of the patch are in flight together, and a tap's
// weights (of 16 channels at a time) are fetched in one go.  Four convs of 16 channels on nine bins of 64 x 64: 37.6 -> 27.4 us a call.
// AHEAD: the patch is requested before the image count is known (conv() below says when).
template <bool U8, int CIN, bool AHEAD>
__global__ __launch_bounds__(256) void k_conv3x3_f32_lds(const void* __restrict__ in_, const float* __restrict__ w4,
                                                         const float* __restrict__ bias, float* out, const float* skip,
                                                         int H, int W, int Cin_, int Cout, int relu, int ps,
                                                         const uint32_t* __restrict__ n_valid, int tiles_x)
{
    extern __shared__ __attribute__((aligned(16))) float patch[];       // [18 * 18][pitch]
    const int n = blockIdx.z, Cin = CIN ? CIN : Cin_;
    if (!AHEAD && n_valid && (uint32_t)n >= *n_valid) return;
    const int tid = threadIdx.x, tyb = blockIdx.x / tiles_x, txb = blockIdx.x - tyb * tiles_x;
    const int x0 = txb * 16, y0 = tyb * 16, pitch = (Cin + 7) & ~3;     // >= Cin + 4: neighbouring pixels start in other banks
    const int co0 = blockIdx.y * CO_L;
    float acc[CO_L];
#pragma unroll
    for (int j = 0; j < CO_L; ++j) acc[j] = bias[min(co0 + j, Cout - 1)];
    if constexpr (CIN != 0) {
        // all of a thread's pieces (float4, or bytes) in flight together
        constexpr int PC = U8 ? CIN : CIN / 4, TOTAL = 18 * 18 * PC, NP = (TOTAL + 255) / 256;
        static_assert(NP <= 11, "pieces in registers");
        using piece = std::conditional_t<U8, uint8_t, float4>;
        const piece* src = (const piece*)in_ + (size_t)n * H * W * PC;
        piece v[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int i = j * 256 + tid, px = i / PC, row = px / 18, gy = y0 - 1 + row, gx = x0 - 1 + px - row * 18;
            v[j] = piece{};
            if (i < TOTAL && gy >= 0 && gy < H && gx >= 0 && gx < W) v[j] = src[((size_t)gy * W + gx) * PC + (i - px * PC)];
        }
        if (AHEAD && n_valid && (uint32_t)n >= *n_valid) return;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int i = j * 256 + tid, px = i / PC;
            if (i < TOTAL) {
                if constexpr (U8) patch[px * pitch + (i - px * PC)] = __fdiv_rn((float)v[j], 255.0f);
                else *(float4*)(patch + px * pitch + (i - px * PC) * 4) = v[j];
            }
        }
    } else if (!U8 && (Cin & 3) == 0) {
        const float4* src = (const float4*)in_;
        const int q = Cin >> 2, total = 18 * 18 * q;
        for (int i0 = 0; i0 < total; i0 += 256 * 6) {
            float4 v[6];
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                const int i = i0 + j * 256 + tid, px = i / q, row = px / 18, gy = y0 - 1 + row, gx = x0 - 1 + px - row * 18;
                v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (i < total && gy >= 0 && gy < H && gx >= 0 && gx < W) v[j] = src[(((size_t)n * H + gy) * W + gx) * q + (i - px * q)];
            }
#pragma unroll
            for (int j = 0; j < 6; ++j) {
                const int i = i0 + j * 256 + tid, px = i / q;
                if (i < total) *(float4*)(patch + px * pitch + (i - px * q) * 4) = v[j];
            }
        }
    } else {
        const int total = 18 * 18 * Cin;
        for (int i = tid; i < total; i += 256) {
            const int px = i / Cin, c = i - px * Cin, row = px / 18, gy = y0 - 1 + row, gx = x0 - 1 + px - row * 18;
            float v = 0.f;
            if (gy >= 0 && gy < H && gx >= 0 && gx < W) {
                const size_t o = (((size_t)n * H + gy) * W + gx) * Cin + c;
                v = U8 ? __fdiv_rn((float)((const uint8_t*)in_)[o], 255.0f) : ((const float*)in_)[o];
            }
            patch[px * pitch + c] = v;
        }
    }
    __syncthreads();
    const int x = x0 + (tid & 15), y = y0 + (tid >> 4);
    if (x >= W || y >= H) return;
    const float4* wb = (const float4*)w4 + (size_t)blockIdx.y * 9 * Cin;
    for (int ky = 0; ky < 3; ++ky) {
        if (y + ky < 1 || y + ky > H) continue;              // zero padding: no tap there
        for (int kx = 0; kx < 3; ++kx) {
            if (x + kx < 1 || x + kx > W) continue;
            const float* p = patch + (((tid >> 4) + ky) * 18 + (tid & 15) + kx) * pitch;
            const float4* wt = wb + (ky * 3 + kx) * Cin;     // uniform
            int ci = 0;
            if constexpr (CIN != 0 && CIN % 16 == 0) {
                for (; ci < CIN; ci += 16) {
                    float wq[16][CO_L], vv[16];
#pragma unroll
                    for (int k = 0; k < 16; ++k) *(float4*)wq[k] = wt[ci + k];
#pragma unroll
                    for (int k = 0; k < 16; k += 4) *(float4*)(vv + k) = *(const float4*)(p + ci + k);
#pragma unroll
                    for (int k = 0; k < 16; ++k)
#pragma unroll
                        for (int j = 0; j < CO_L; ++j) acc[j] = fmaf(wq[k][j], vv[k], acc[j]);
                }
                continue;
            }
            for (; ci + 4 <= Cin; ci += 4) {
                const float4 v = *(const float4*)(p + ci);
                const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float4 wv = wt[ci + k];
                    acc[0] = fmaf(wv.x, vv[k], acc[0]); acc[1] = fmaf(wv.y, vv[k], acc[1]);
                    acc[2] = fmaf(wv.z, vv[k], acc[2]); acc[3] = fmaf(wv.w, vv[k], acc[3]);
                }
            }
            for (; ci < Cin; ++ci) {
                const float4 wv = wt[ci]; const float v = p[ci];
                acc[0] = fmaf(wv.x, v, acc[0]); acc[1] = fmaf(wv.y, v, acc[1]); acc[2] = fmaf(wv.z, v, acc[2]); acc[3] = fmaf(wv.w, v, acc[3]);
            }
        }
    }
    if (ps == 1 && (Cout & 3) == 0) {                        // a whole 16-byte piece of the pixel
        const size_t o = (((size_t)n * H + y) * W + x) * Cout + co0;
        float4 r = make_float4(acc[0], acc[1], acc[2], acc[3]);
        if (relu) { r.x = fmaxf(r.x, 0.0f); r.y = fmaxf(r.y, 0.0f); r.z = fmaxf(r.z, 0.0f); r.w = fmaxf(r.w, 0.0f); }
        if (skip) { const float4 s = *(const float4*)(skip + o); r.x += s.x; r.y += s.y; r.z += s.z; r.w += s.w; }
        *(float4*)(out + o) = r;
        return;
    }
    const int r2 = ps * ps, Co = Cout / r2;
#pragma unroll
    for (int j = 0; j < CO_L; ++j) {
        const int co = co0 + j;
        if (co >= Cout) break;
        float v = acc[j];
        if (relu) v = fmaxf(v, 0.0f);
        const int c = co / r2, sub = co - c * r2, si = sub / ps, sj = sub - si * ps;
        const size_t o = (((size_t)n * H * ps + (size_t)y * ps + si) * (W * ps) + (size_t)x * ps + sj) * Co + c;
        if (skip) v += skip[o];
        out[o] = v;
    }
}

// [co / 4][tap][ci][4] copies of the layers with at most LDS_CIN input channels; they lie behind the blob
void rh_pack_weights_f32(rh_ctx* ctx, const float* blob, size_t n_floats, std::vector<float>& packed)
{
    for (rh_layer& L : ctx->layers) {
        if (L.cin > LDS_CIN) continue;
        packed.resize(packed.size() + (0 - n_floats - packed.size()) % 4);       // 16-byte pieces
        L.wp_off = n_floats + packed.size();
        const int nb = (L.cout + CO_L - 1) / CO_L;
        for (int b = 0; b < nb; ++b)
            for (int tap = 0; tap < 9; ++tap)
                for (int ci = 0; ci < L.cin; ++ci)
                    for (int j = 0; j < CO_L; ++j) {
                        const int co = b * CO_L + j;
                        packed.push_back(co < L.cout ? blob[L.w_off + ((size_t)co * 9 + tap) * L.cin + ci] : 0.0f);
                    }
    }
}

static void conv(rh_ctx* ctx, const rh_layer& L, const void* in, int in_u8, float* out, const float* skip,
                 int N, int H, int W, int relu, int ps, const uint32_t* n_valid)
{
    const int tiles_x = (W + 15) / 16, tiles_y = (H + 15) / 16;
    if (L.cin <= LDS_CIN) {
        static bool attr_done[RH_MAX_DEVICES] = {};          // the attribute is per device
        if (!attr_done[ctx->device])
            attr_done[ctx->device] = hipFuncSetAttribute((const void*)k_conv3x3_f32_lds<false, 0, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                         18 * 18 * (LDS_CIN + 4) * sizeof(float)) == hipSuccess;
        const dim3 grid(tiles_x * tiles_y, (L.cout + CO_L - 1) / CO_L, N);
        const size_t lds = (size_t)18 * 18 * ((L.cin + 7) & ~3) * sizeof(float);
        const float* w4 = ctx->w_f32 + L.wp_off;
        // Ahead of the count where the grid is small enough to run at once: then images that are not valid cost no time.  In a larger one their
        // patches do.  us a call, ahead / behind the count, 4 convs of 16 channels on 9 valid of N bins of 64 x 64 (64 workgroups each): N = 9
        // 27.3 / 28.1, 32: 26.6 / 27.8, 64: 31.2 / 27.7, 400: 101 / 31; residual net of 32 channels on 4 valid of N of 96 x 96 (288 each): 4
        // 117.4 / 119.2, 16: 122.3 / 119.4, 64: 254 / 122; all 64 bins of 64 x 64 valid 87.1 / 88.5.  The line is at 8 workgroups a CU.
        const bool ahead = (long long)grid.x * grid.y * grid.z <= 8ll * ctx->n_cu;
#define KERN(U8, CIN) (ahead ? k_conv3x3_f32_lds<U8, CIN, true> : k_conv3x3_f32_lds<U8, CIN, false>)
        auto kern = in_u8 ? (L.cin == 3 ? KERN(true, 3) : k_conv3x3_f32_lds<true, 0, false>)
                          : (L.cin == 16 ? KERN(false, 16) : L.cin == 32 ? KERN(false, 32) : k_conv3x3_f32_lds<false, 0, false>);
#undef KERN
        hipLaunchKernelGGL(kern, grid, dim3(256), lds, ctx->stream, in, w4, ctx->w_f32 + L.b_off, out, skip, H, W, L.cin, L.cout, relu, ps, n_valid, tiles_x);
        return;
    }
    hipLaunchKernelGGL(k_conv3x3_f32, dim3(tiles_x * tiles_y, (L.cout + CO_T - 1) / CO_T, N), dim3(256), 0,
                       ctx->stream, in, in_u8, ctx->w_f32 + L.w_off, ctx->w_f32 + L.b_off, out, skip, H, W, L.cin,
                       L.cout, relu, ps, n_valid, tiles_x);
}

rh_status rh_launch_enhance_fp32(rh_ctx* ctx, const uint8_t* in, int N, int H, int W, float* out,
                                 const uint32_t* n_valid)
{
    const rh_net_desc& d = ctx->cfg.net;
    const int C = d.channels, s = d.scale;
    const size_t lr = (size_t)N * H * W * C;
    size_t need = 3 * lr;
    size_t up1 = 0, up2 = 0;
    if (d.topology == RH_NET_EDSR) {
        const int r = (s == 4) ? 2 : s;
        up1 = lr * r * r; need += up1;
        if (s == 4) { up2 = up1 * 4; need += up2; }
    }
    rh_status st = rh_ensure_workspace(ctx, need * sizeof(float));
    if (st != RH_OK) return st;
    float* a = (float*)ctx->act; float* t = a + lr; float* h = t + lr; float* u1 = h + lr; float* u2 = u1 + up1;
    const std::vector<rh_layer>& L = ctx->layers;
    size_t li = 0;
    const uint32_t nl = (uint32_t)L.size();
    rh_prof_scope ps(ctx, RH_PROF_CONV, ctx->bz_boxes ? 2 * nl - 1 : nl);       // all layers of the fp32 path count as one class
    // exact-border mode (a no-op otherwise): clear the out-of-frame part of the boxes in a layer's output
#define ZERO(buf, res) do { st = rh_zero_outside(ctx, (buf), C * (int)sizeof(float), (res), N, n_valid); if (st != RH_OK) return st; } while (0)
    if (d.topology == RH_NET_PLAIN) {
        conv(ctx, L[li++], in, 1, a, nullptr, N, H, W, 1, 1, n_valid); ZERO(a, 1);
        for (int l = 0; l < d.n_blocks - 2; ++l) { conv(ctx, L[li++], a, 0, t, nullptr, N, H, W, 1, 1, n_valid); ZERO(t, 1); float* sw = a; a = t; t = sw; }
        conv(ctx, L[li++], a, 0, out, nullptr, N, H, W, 0, s, n_valid);
    } else {
        conv(ctx, L[li++], in, 1, h, nullptr, N, H, W, 0, 1, n_valid); ZERO(h, 1);
        const float* x = h;                         // block input; the head output stays in h for EDSR
        for (int b = 0; b < d.n_blocks; ++b) {
            conv(ctx, L[li++], x, 0, t, nullptr, N, H, W, 1, 1, n_valid); ZERO(t, 1);
            // x + conv(t): for the first block the result goes to a so that h survives
            conv(ctx, L[li++], t, 0, a, x, N, H, W, 0, 1, n_valid); ZERO(a, 1);
            x = a;
        }
        if (d.topology == RH_NET_RES) {
            conv(ctx, L[li++], x, 0, out, nullptr, N, H, W, 0, s, n_valid);
        } else {
            conv(ctx, L[li++], x, 0, t, h, N, H, W, 0, 1, n_valid); ZERO(t, 1);         // body end + long skip
            const int r = (s == 4) ? 2 : s;
            conv(ctx, L[li++], t, 0, u1, nullptr, N, H, W, 0, r, n_valid); ZERO(u1, r);
            const float* last = u1; int hh = H * r, ww = W * r;
            if (s == 4) { conv(ctx, L[li++], u1, 0, u2, nullptr, N, hh, ww, 0, 2, n_valid); ZERO(u2, 2 * r); last = u2; hh *= 2; ww *= 2; }
            conv(ctx, L[li++], last, 0, out, nullptr, N, hh, ww, 0, 1, n_valid);
        }
    }
#undef ZERO
    RH_HIP(ctx, hipGetLastError());
    return RH_OK;
}
