// The upsampler and the last conv of the EDSR-shaped nets as ONE convolution (Sec. 3.3.3: the
// enhancement model applied to the packed bins).
//
// After the body, these nets are linear: conv C -> C*r*r, pixel shuffle (once, or twice by 2 for
// x4), conv C -> 3, with no activation in between.  A composition of linear maps is a linear map:
// every output pixel (s*y + i, s*x + j) is a bias plus a weighted sum over the 5 x 5 neighbourhood
// of low-resolution pixel (y, x) of the body's output t,
//     out[s*y+i][s*x+j][co] = B[i][j][co] + sum_{dy,dx in -2..2} sum_ci Wc[i][j][co][dy][dx][ci] * t[y+dy][x+dx][ci],
// i.e. a 5 x 5 convolution C -> 3*s*s at low resolution followed by a pixel shuffle.  Executed
// that way the high-resolution 64-channel tensors (2.4 GB written and read back per batch at x4)
// never exist and the arithmetic shrinks about sevenfold.
//
// Wc and B are computed once at rh_create (in double, from the given weights) by pushing the
// gradient of each output through the layers, then rounded to bf16 for the matrix cores.  The
// layers pad with zeros at their own tensor's border, so the intermediate tensors outside the
// image are zero, not "what the previous conv would give there": Wc differs for the pixels of the
// outermost low-resolution ring.  There are 9 position classes (top / middle / bottom row x left
// / middle / right column); the interior is computed with the middle class, the ring pixel by pixel with the
// weights of its class.
//
// Main kernel: implicit GEMM on v_mfma_f32_16x16x32_bf16, D[row][pixel], rows = (i, j, co) in tiles of 16 (x4: 48 rows in three, x3: 27 in two, x2: 12 in
// one), N = 16 pixels of an image row, K = tap * C + ci over 25 taps.  One persistent workgroup per CU works on 8 x 32 pixels, from a
// 12 x 36 pixel patch in LDS (same channels-last layout and XOR swizzle as the 3 x 3 kernels), the next one's copied meanwhile.  A wave has one tile of
// rows, 32 of C and a part of the pixels: its 25 weight fragments stay in registers, and an activation fragment, read once, feeds the up to five
// image rows that it belongs to.  64 channels: the two waves that share rows and pixels exchange half of their sums each.  The sums go through LDS
// in the order of the output, so that stores are whole lines: 16 bytes a lane, 4 where an image row's start or the ring cuts a group of four.
// What bounds it: instruction issue (x4, an 8 x 32 tile: 9 600 cycles of products, 17 000 in all; a product of 16 cycles hides two other instructions).
// With 32-row tiles (two at x4, three quarters full; one at x2, 3/8 full), a quarter of C a wave, all partial sums exchanged, and stores straight from
// the sums, 4 bytes a lane at x3, then / now: the kernel on 76 bins of 128 x 128 x4 280 / 182 us, 264 bins x3 880 / 655; whole steps, the headline batch
// 2 540 / 2 470, 16 whole frames 4 490 / 4 390, 32 frames 640 x 368 x3 9 900 / 9 790.
#include <string.h>

#include <atomic>
#include <new>
#include <thread>
#include <type_traits>

#include "conv_mfma_common.h"

#define FOLD_TH 8
#define FOLD_PW 36

struct fold_args {
    const __bf16* in;        // t: [N][H][W][CIN]
    const uint4* wp;         // [class][chunk][tap][ks][lane]; middle class: [tap][32 of C][16 rows][lane]
    const float* bias;       // [class][chunk][32]; middle class: by row
    float* out;              // [N][s*H][s*W][3]
    const uint32_t* n_valid;
    int N, H, W;
    int n_chunks;            // of the ring's weights: 32 rows each
    int rev;
    int ring;                // 1: the outermost ring with its classes' weights; 0: it is not needed (no pixel of it is pasted)
    const uint32_t* tile_list;   // the tiles to compute (needed-region mode), or null: all tiles
    const uint32_t* n_list;
};

// Stores the 16 accumulator values of one lane: rows 8q + 4hi + e of chunk `chunk` for
// low-resolution pixel (y, x) of image n.  Row rho of a chunk is (il, j, co) = (rho / 3s, rho / 3 % s,
// rho % 3) with output row i = chunk * ipc + il.
template <int s>
__device__ __forceinline__ void fold_store(const fold_args& a, const f32x16& acc, int n, int y, int x, int chunk, int hi)
{
    const int OW = a.W * s;
    float* base = a.out + (((size_t)n * a.H * s + (size_t)y * s) * OW + (size_t)x * s) * 3;
    if (s == 4) {                      // 12 values per output row i: three aligned groups of four
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int rho = 8 * q + 4 * hi, il = rho / 12, off = rho - 12 * il;
            *(float4*)(base + (size_t)(chunk * 2 + il) * OW * 3 + off) = make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
        }
        return;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int rho = 8 * q + 4 * hi + e;
            if (rho >= 3 * s * s) continue;
            const int il = rho / (3 * s), rem = rho - il * 3 * s;
            base[(size_t)(chunk * s + il) * OW * 3 + rem] = acc[4 * q + e];
        }
}

template <int N, int I = 0, typename F>
__device__ __forceinline__ void fold_each_step(F& f)
{
    if constexpr (I < N) { f(std::integral_constant<int, I>{}); fold_each_step<N, I + 1>(f); }
}

// The outermost ring of every image, with the weights of its position class: wave `w` of `waves` takes every waves-th group of
// 32 ring pixels and chunk, operands straight from global memory (the ring is 3 % of the pixels).
// Classes are numbered 3 * (0 top / 1 middle / 2 bottom) + (0 left / 1 middle / 2 right).
// Two rows of taps of an edge pixel lie outside the image (or two columns): 15 taps of 25 are left, 9 at a corner, three in flight.
// A launch of its own behind the main kernel took 45 us on 76 bins of 128 x 128 and 9 on three; as the work that the main
// kernel's waves do when they are out of tiles (idle workgroups at once): whole calls of EDSR x3 with one block on three bins 59.6 -> 51.6 us,
// x4 on 76 566 -> 563, on 128 943 -> 938, on 16 of 64 x 64 60.0 -> 60.6.
template <int CIN, int S>
__device__ __forceinline__ void fold_ring(const fold_args& a, int n_img, long w, long waves)
{
    constexpr int KS = CIN / 16;
    const int lane = threadIdx.x & 63, lx = lane & 31, hi = lane >> 5;
    const long row_g = ((long)n_img * (a.W - 2) + 31) / 32, col_g = ((long)n_img * (a.H - 2) + 31) / 32, corner_g = (n_img + 31) / 32;
    const long groups = 2 * row_g + 2 * col_g + 4 * corner_g;
    for (long u = w; u < groups * a.n_chunks; u += waves) {      // uniform over the wave
        const int chunk = (int)(u / groups);
        long g = u - chunk * groups;
        int kind = 0;                                        // top, bottom, left, right edges, then the corners
        for (long size; g >= (size = kind < 2 ? row_g : kind < 4 ? col_g : corner_g); ++kind) g -= size;
        const int per = kind < 2 ? a.W - 2 : kind < 4 ? a.H - 2 : 1;      // ring pixels of this class per image
        const bool top = kind == 0 || kind == 4 || kind == 5, bottom = kind == 1 || kind >= 6;
        const bool left = kind == 2 || kind == 4 || kind == 6, right = kind == 3 || kind == 5 || kind == 7;
        const int cls = (top ? 0 : bottom ? 6 : 3) + (left ? 0 : right ? 2 : 1);
        const long q = g * 32 + lx;
        const bool valid = q < (long)n_img * per;
        const int n = valid ? (int)(q / per) : 0, k = valid ? (int)(q - (long)n * per) : 0;
        const int y = top ? 0 : bottom ? a.H - 1 : 1 + k, x = left ? 0 : right ? a.W - 1 : 1 + k;
        const uint4* wp = a.wp + (size_t)(cls * a.n_chunks + chunk) * (25 * KS * 64);
        const float* bias = a.bias + (cls * a.n_chunks + chunk) * 32;
        f32x16 acc;
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = bias[(e >> 2) * 8 + hi * 4 + (e & 3)];
        const __bf16* img = a.in + (size_t)n * a.H * a.W * CIN;
        const int ky0 = top ? 2 : 0, kx0 = left ? 2 : 0, nkx = kind < 2 ? 5 : 3, taps = kind < 4 ? 15 : 9;
        uint4 A[3][KS], B[3][KS];
        auto load_tap = [&](int t, uint4 (&At)[KS], uint4 (&Bt)[KS]) __attribute__((always_inline)) {
            const int ky = ky0 + t / nkx, kx = kx0 + t % nkx, yy = y + ky - 2, xx = x + kx - 2;
            const bool ok = valid && yy >= 0 && yy < a.H && xx >= 0 && xx < a.W;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                At[ks] = wp[((ky * 5 + kx) * KS + ks) * 64 + lane];
                Bt[ks] = ok ? *(const uint4*)(img + ((size_t)yy * a.W + xx) * CIN + ks * 16 + hi * 8) : make_uint4(0, 0, 0, 0);
            }
        };
#pragma unroll
        for (int t = 0; t < 3; ++t) load_tap(t, A[t], B[t]);
        for (int t0 = 0; t0 < taps; t0 += 3) {
#pragma unroll
            for (int t = 0; t < 3; ++t) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*(const bf16x8*)&A[t][ks], *(const bf16x8*)&B[t][ks], acc, 0, 0, 0);
                load_tap(min(t0 + t + 3, taps - 1), A[t], B[t]);
            }
        }
        if (valid) fold_store<S>(a, acc, n, y, x, chunk, hi);
    }
}

// What a wave of the main kernel has: one of MT tiles of 16 rows, one of KH halves of C, one of PG parts of the 8 x 32 pixels - R image rows, 16 columns.
template <int CIN, int S>
struct fold_shape {
    static constexpr int MT = (3 * S * S + 15) / 16, KH = CIN / 32, PG = MT * KH >= 4 ? 2 : MT * KH >= 2 ? 4 : 8, WAVES = MT * KH * PG, R = 16 / PG;
    static constexpr int PASSES = KH == 2 && WAVES > 8 ? 2 : 1;      // three waves a SIMD: registers for half of the rows' sums
    static constexpr int PATCHB = (FOLD_TH + 4) * FOLD_PW * CIN * 2, OUT = FOLD_TH * S * 96 * S * 4, LDS = 2 * PATCHB + OUT;
    static_assert(PATCHB % 1024 == 0 && LDS + KH * MT * 64 <= 160 * 1024, "a patch is whole pieces; all of it fits");
};

// C of a lane's four sums, from the e-th on, to and from LDS; `at` is aligned to C floats
template <int C, int e>
__device__ __forceinline__ void fold_put(float* at, const f32x4& v)
{
    if constexpr (C == 4) *(float4*)at = make_float4(v[0], v[1], v[2], v[3]);
    else if constexpr (C == 2) *(float2*)at = make_float2(v[e], v[e + 1]);
    else *at = v[e];
}
template <int C, int e>
__device__ __forceinline__ void fold_get(f32x4& v, const float* at)
{
    if constexpr (C == 4) { const float4 f = *(const float4*)at; v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w; }
    else if constexpr (C == 2) { const float2 f = *(const float2*)at; v[e] = f.x; v[e + 1] = f.y; }
    else v[e] = *at;
}

template <int CIN, int S, bool LIST>
__global__ __launch_bounds__((fold_shape<CIN, S>::WAVES * 64)) void k_conv_fold(fold_args a)
{
    // LIST: the tiles come from a.tile_list.  An entry is requested two tiles ahead with a vector
    // load (a scalar load would share its counter with the LDS fragment reads) and read a tile later.
    using L = fold_shape<CIN, S>;
    constexpr int NCH = CIN / 8, PIXB = CIN * 2, TH = FOLD_TH, PW = FOLD_PW, R = L::R, MT = L::MT, KH = L::KH, W_ = L::WAVES;
    constexpr int RP = L::PASSES == 2 ? R / 2 : R, NFRAG = 5 * (RP + 4);             // image rows of a pass, and its fragments
    constexpr int NPIECE = L::PATCHB / 1024, NPRE = (NPIECE + W_ - 1) / W_;          // a wave's 1 KB pieces of the patch
    constexpr int SWZ_SH = (NCH == 8) ? 0 : 1, PXF = 3 * S, LINE = 32 * PXF;         // output floats of a pixel's and of the tile's image row
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    float* lds_o = (float*)(lds + 2 * L::PATCHB);                                    // [8 S lines][LINE]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = wave % MT, kh = wave / MT % KH, pg = wave / (MT * KH);
    const int col0 = (pg & 1) * 16, row0 = (pg >> 1) * R;                            // of the wave's pixels

    const uint32_t* counter = LIST ? a.n_list : a.n_valid;
    const uint32_t n_found = counter ? *counter : (uint32_t)a.N;
    // the weights and the bias are on their way before the image count is known
    const uint4* wp = a.wp + (size_t)4 * a.n_chunks * 25 * (CIN / 16) * 64 + (kh * MT + m) * 64 + lane;      // the middle class
    bf16x8 A[25];
#pragma unroll
    for (int t = 0; t < 25; ++t) A[t] = *(const bf16x8*)(wp + t * (KH * MT * 64));
    // The bias, in the sums of the first half of C, is read from LDS for every tile: three waves a SIMD have few registers to spare.  With the bias kept over
    // the loop / with this, whole calls with one block on 16 of 64 x 64, 32 channels, us, x2 38.9 / 36.0, x4 42.5 / 40.3; others level.
    __shared__ __attribute__((aligned(16))) float s_bias[KH][16 * MT];
    if (tid < KH * 16 * MT) s_bias[0][tid] = tid < 16 * MT ? a.bias[4 * a.n_chunks * 32 + tid] : 0.0f;
    // XCD-contiguous tile runs, as in the 3 x 3 kernels
    const int G = gridDim.x;
    const int wg = (G % 8 == 0) ? (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8 : (int)blockIdx.x;
    const int n_img = min((int)n_found, a.N);
    const int tiles_x = (a.W + 31) / 32, tiles_y = (a.H + TH - 1) / TH, tiles_img = tiles_x * tiles_y;
    const int n_tiles = LIST ? (int)n_found : n_img * tiles_img;
    const uint32_t in_img_bytes = (uint32_t)a.H * a.W * PIXB;

    // piece i of the patch, by wave i % WAVES: 64 16-byte channel groups, 8 (16) pixels.  The pieces are contiguous in LDS, so the
    // lanes fetch swizzled.  Rows outside the image lie outside the descriptor's range and read as zeros.  (Inline asm, with no register written: behind
    // the builtin the compiler has LDS accesses wait for the copy.)
    // (`l` is the lane, passed through an empty asm statement in every phase: addresses kept over the loop would not fit the registers.)
    auto lane_now = [&]() __attribute__((always_inline)) { int l = lane; asm volatile("" : "+v"(l)); return l; };
    auto load_patch = [&](uint8_t* to, __amdgpu_buffer_rsrc_t rin, int y0, int x0) __attribute__((always_inline)) {
        const int l = lane_now();
#pragma unroll
        for (int j = 0; j < NPRE; ++j) {
            const int i = j * W_ + wave;
            if (j == NPRE - 1 && i >= NPIECE) break;
            const uint32_t idx = i * 64 + l, px = idx / NCH, row = (px * 1821u) >> 16, col = px - row * PW;      // px / 36 for px < 432
            const int gx = x0 - 2 + (int)col;
            const uint32_t off = (uint32_t)((y0 - 2 + (int)row) * a.W + gx) * PIXB + (((idx ^ (col >> SWZ_SH)) & (NCH - 1)) << 4);
            const uint32_t at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)(to + i * 1024));
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                         :: "s"(at), "v"((uint32_t)gx < (uint32_t)a.W ? off : OOB_OFF), "s"(rin) : "memory", "m0");
        }
    };
    __amdgpu_buffer_rsrc_t rlist = __builtin_amdgcn_make_buffer_rsrc((void*)a.tile_list, 0, LIST ? (uint32_t)n_tiles * 4u : 0u, RSRC_FLAGS);
    auto list_load = [&](int idx) __attribute__((always_inline)) {       // entry of walk position idx (0 past the end)
        const int pos = a.rev ? n_tiles - 1 - idx : idx;
        return __builtin_amdgcn_raw_buffer_load_b32(rlist, idx < n_tiles ? (uint32_t)pos * 4u : OOB_OFF, 0, 0);
    };
    auto decode_cell = [&](int cell, int& n, int& y0, int& x0) __attribute__((always_inline)) {    // RH_CELL_ENTRY
        n = (int)((uint32_t)cell >> 16); y0 = (int)(((uint32_t)cell >> 7) & 511u) * TH; x0 = (int)((uint32_t)cell & 127u) * 32;
    };
    auto tile_origin = [&](int tile, int& n, int& y0, int& x0) __attribute__((always_inline)) {
        if constexpr (LIST) { decode_cell(__builtin_amdgcn_readfirstlane(list_load(tile)), n, y0, x0); return; }
        if (a.rev && tile < n_tiles) tile = n_tiles - 1 - tile;          // walk back over what the previous layer wrote last
        n = tile / tiles_img;
        const int tr = tile - n * tiles_img, ty = tr / tiles_x;
        y0 = ty * TH; x0 = (tr - ty * tiles_x) * 32;
    };
    auto in_rsrc = [&](int tile, int n) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)(a.in + (size_t)n * a.H * a.W * CIN), 0,
                                                 tile < n_tiles ? in_img_bytes : 0u, RSRC_FLAGS);
    };
    // four rows of sums of a pixel, and their places in the tile's output: LINE floats a line, of which the pixel has 3 S in each of S lines
    auto places = [&](auto&& put) __attribute__((always_inline)) {       // put(first of the rows, how many, where)
        const int l = lane_now(), rho = m * 16 + (l >> 4) * 4, px = (l & 15) + col0;
        constexpr int STEP = S == 4 ? 4 : S == 2 ? 2 : 1;
        auto part = [&](auto k_c) __attribute__((always_inline)) {
            constexpr int e = decltype(k_c)::value * STEP;
            const int i = (rho + e) / PXF;
            if (S == 4 || rho + e < S * PXF) put(std::integral_constant<int, STEP>{}, std::integral_constant<int, e>{}, lds_o + row0 * S * LINE + i * LINE + px * PXF + (rho + e - i * PXF));
        };
        fold_each_step<4 / STEP>(part);
    };

    // the tile's output, whole in LDS, to memory; n < 0: there is none
    auto store = [&](int n, int y0, int x0) __attribute__((always_inline)) {
        if (n < 0) return;
        const int off = a.ring;                            // the ring's pixels are another wave's
        const int lo = off && x0 == 0 ? PXF : 0, hi = min(32, a.W - off - x0) * PXF, pitch = a.W * PXF;
        float* base = a.out + (((size_t)n * a.H + y0) * S) * pitch + x0 * PXF;
        const int lines0 = off && y0 == 0 ? S : 0, lines1 = min(TH, a.H - off - y0) * S;
        const int t = wave * 64 + lane_now();
        if (S == 4 || (pitch & 3) == 0) {
#pragma unroll
            for (int u0 = 0; u0 < TH * S * LINE / 4; u0 += W_ * 64) {
                const int u = u0 + t, line = u / (LINE / 4), col = (u - line * (LINE / 4)) * 4;
                if (u0 + W_ * 64 > TH * S * LINE / 4 && u >= TH * S * LINE / 4) break;
                const float4 v = *(const float4*)(lds_o + u * 4);
                float* to = base + (size_t)line * pitch + col;
                if (line < lines0 || line >= lines1) continue;
                if (S == 4 ? col >= lo && col < hi : col >= lo && col + 4 <= hi) { *(float4*)to = v; continue; }
                if constexpr (S != 4) {                    // the ring or the image's end cuts the four
                    if (col >= lo && col < hi) to[0] = v.x;
                    if (col + 1 >= lo && col + 1 < hi) to[1] = v.y;
                    if (col + 2 >= lo && col + 2 < hi) to[2] = v.z;
                    if (col + 3 >= lo && col + 3 < hi) to[3] = v.w;
                }
            }
        } else {
#pragma unroll 4
            for (int u = t; u < TH * S * LINE; u += W_ * 64) {
                const int line = u / LINE, col = u - line * LINE;
                const float v = lds_o[u];
                if (line >= lines0 && line < lines1 && col >= lo && col < hi) base[(size_t)line * pitch + col] = v;
            }
        }
    };
    int n, y0, x0, e_next = 0;
    tile_origin(wg, n, y0, x0);
    if constexpr (LIST) e_next = list_load(wg + G);
    load_patch(lds, in_rsrc(wg, wg < n_tiles ? n : 0), y0, x0);
    lds_dma_wait();                                        // and the weights
    lds_barrier();
    uint8_t* patch = lds;
    int nn = n, ny0 = y0, nx0 = x0, pn = -1, py0 = 0, px0 = 0;       // origins of the next and of the last tile
    for (int tile = wg; tile < n_tiles; tile += G) {       // trip count uniform over the workgroup
        uint8_t* other = patch == lds ? lds + L::PATCHB : lds;
        // what is to be done beside the products
        auto aside = [&]() __attribute__((always_inline)) {
            store(pn, py0, px0);
            const int nt = tile + G;
            if constexpr (LIST) { const int e_after = list_load(tile + 2 * G); decode_cell(__builtin_amdgcn_readfirstlane(e_next), nn, ny0, nx0); e_next = e_after; }
            else tile_origin(nt, nn, ny0, nx0);
            load_patch(other, in_rsrc(nt, nt < n_tiles ? nn : 0), ny0, nx0);
        };

        // RP rows of pixels from patch row `prow` on.  Fragment i: tap column i / (RP + 4), image row i % (RP + 4); two at a time, read a pair ahead.  Two
        // sums a row, of the taps of a chessboard's colours (three waves a SIMD, where that does not fit the registers: of even and of odd tap columns): with
        // the halves of C four chains of products.  In one chain a half of C the error against 64 bits was a third larger; so it is what it was with a
        // quarter of C in each of four waves (64 channels, rms at x2, x3, x4: 4.5, 4.0, 6.6e-9 of 0.055; 4.8, 4.3, 6.7 then).
        f32x4 acc[2][RP];
        bf16x8 B[4];
        auto pass = [&](const uint8_t* prow, auto between) __attribute__((always_inline)) {
            const int l = lane_now();
            auto load = [&](int i) __attribute__((always_inline)) {
                const int px = col0 + (l & 15) + i / (RP + 4);
                B[i % 4] = *(const bf16x8*)(prow + px * PIXB + (((4 * kh + (l >> 4)) ^ ((px >> SWZ_SH) & (NCH - 1))) << 4) + i % (RP + 4) * (PW * PIXB));
            };
            const f32x4 bias_c = *(const f32x4*)(s_bias[kh] + m * 16 + (l >> 4) * 4);      // of rows 16 m + 4 (lane / 16) + {0..3}
            load(0); load(1);
            __builtin_amdgcn_sched_barrier(0);
            auto frag = [&](auto i_c) __attribute__((always_inline)) {
                constexpr int i = decltype(i_c)::value, kx = i / (RP + 4), py = i % (RP + 4), k0 = py < RP ? 0 : py - RP + 1, k1 = py < 4 ? py : 4;
                if constexpr (i % 2 == 0) asm volatile("" :: "v"(B[i % 4]), "v"(B[(i + 1) % 4]));
#pragma unroll
                for (int k = 0; k <= k1 - k0; ++k) {       // there and back over the rows: from one product to the next only one operand changes
                    const int ky = i % 2 ? k1 - k : k0 + k;
                    const int set = (W_ > 8 ? kx : kx + ky) & 1, first = W_ > 8 ? ky == 0 && kx < 2 : kx == 0 && ky < 2;
                    f32x4& d = acc[set][py - ky];
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[ky * 5 + kx], B[i % 4], !first ? d : set ? f32x4{0, 0, 0, 0} : bias_c, 0, 0, 0);
                    if (k == 0 && i + 2 < NFRAG) load(i + 2);
                    __builtin_amdgcn_sched_barrier(0);
                }
                between(i_c);
            };
            fold_each_step<NFRAG>(frag);
#pragma unroll
            for (int r = 0; r < RP; ++r)
#pragma unroll
                for (int z = 0; z < 4; ++z) acc[0][r][z] += acc[1][r][z];
        };
        auto nothing = [](auto) {};
        auto with_aside = [&](auto i_c) __attribute__((always_inline)) {
            // in the waves of a SIMD one after the other, so that the others keep the matrix pipe busy
            constexpr int i = decltype(i_c)::value, D = NFRAG / (L::PASSES == 2 ? 4 : 6);
            if constexpr (i >= 2 && (i - 2) % D == 0 && (i - 2) / D < W_ / 4) if (wave / 4 == (i - 2) / D) aside();
            if constexpr (L::PASSES == 1 && i == NFRAG / 2) asm volatile("s_barrier" ::: "memory");       // every wave has read the last tile's output from LDS
        };
        // 64 channels: of half of its rows a wave hands its sums over, of the others it adds up both halves of C
        auto put = [&](int row, auto first_c, auto rows_c) __attribute__((always_inline)) {
            places([&](auto c, auto e_c, float* to) __attribute__((always_inline)) {
#pragma unroll
                for (int r = 0; r < decltype(rows_c)::value; ++r) fold_put<decltype(c)::value, decltype(e_c)::value>(to + (row + r) * S * LINE, acc[0][decltype(first_c)::value + r]);
            });
        };
        auto add = [&](int row, auto first_c, auto rows_c) __attribute__((always_inline)) {
            places([&](auto c, auto e_c, float* to) __attribute__((always_inline)) {
                constexpr int C = decltype(c)::value, e = decltype(e_c)::value, N = decltype(rows_c)::value;
                f32x4 v[N];
#pragma unroll
                for (int r = 0; r < N; ++r) fold_get<C, e>(v[r], to + (row + r) * S * LINE);
#pragma unroll
                for (int r = 0; r < N; ++r) {
#pragma unroll
                    for (int z = e; z < e + C; ++z) v[r][z] += acc[0][decltype(first_c)::value + r][z];
                    fold_put<C, e>(to + (row + r) * S * LINE, v[r]);
                }
            });
        };
        constexpr std::integral_constant<int, 0> ZERO{};
        constexpr std::integral_constant<int, KH == 2 ? R / 2 : R> HALF{};
        const uint8_t* rows = patch + row0 * (PW * PIXB);
        const int own = kh * HALF;
        if constexpr (L::PASSES == 2) {
            pass(rows + (HALF - own) * (PW * PIXB), with_aside);
            asm volatile("s_barrier" ::: "memory");        // every wave has read the last tile's output from LDS
            put(HALF - own, ZERO, HALF);
            pass(rows + own * (PW * PIXB), nothing);
            lds_barrier();
            lds_dma_wait();                                // the next patch
            add(own, ZERO, HALF);
        } else {
            pass(rows, with_aside);
            if constexpr (KH == 2) {
                if (kh) put(0, ZERO, HALF); else put(HALF, HALF, HALF);
                lds_barrier();
            }
            lds_dma_wait();
            if constexpr (KH == 1) put(0, ZERO, HALF);
            else if (kh) add(HALF, HALF, HALF);
            else add(0, ZERO, HALF);
        }
        lds_barrier();                                     // the tile's output and the next patch are there
        pn = n; py0 = y0; px0 = x0;
        n = nn; y0 = ny0; x0 = nx0;
        patch = other;
    }
    store(pn, py0, px0);
    if (a.ring) {
        // workgroups that have had a tile more, or one at all, come last
        const int n_ring = a.n_valid ? min((int)*a.n_valid, a.N) : a.N;
        fold_ring<CIN, S>(a, n_ring, (long)((int)gridDim.x - 1 - wg) + (long)wave * gridDim.x, (long)W_ * gridDim.x);
    }
}

// ------------------------------------------------------------------------------------------
// host side: composition of the layers' weights

namespace {

struct fold_stage { const float* w; const float* b; int cin, cout, r; };   // conv3x3 cin -> cout, then pixel shuffle by r

// Gradient of output (Yf, Xf, co) of the last stage's conv with respect to the first stage's input,
// on a small image whose first-stage grid is g0 x g0 (zero padding at every stage's own border).
// grid[k] = side of stage k's input grid.
void fold_gradient(const std::vector<fold_stage>& st, const std::vector<int>& grid, int Yf, int Xf, int co,
                   std::vector<double>& g_in0)
{
    const int K = (int)st.size();
    std::vector<double> gc((size_t)grid[K - 1] * grid[K - 1] * st[K - 1].cout, 0.0);
    gc[((size_t)Yf * grid[K - 1] + Xf) * st[K - 1].cout + co] = 1.0;
    int cy0 = Yf, cy1 = Yf, cx0 = Xf, cx1 = Xf;            // bounding box of the non-zeros of gc
    for (int k = K - 1; k >= 0; --k) {
        const fold_stage& S = st[k];
        const int g = grid[k];
        std::vector<double> gi((size_t)g * g * S.cin, 0.0);
        for (int y = cy0; y <= cy1; ++y) for (int x = cx0; x <= cx1; ++x) for (int c = 0; c < S.cout; ++c) {
            const double v = gc[((size_t)y * g + x) * S.cout + c];
            if (v == 0.0) continue;
            for (int ky = 0; ky < 3; ++ky) {
                const int iy = y + ky - 1; if (iy < 0 || iy >= g) continue;      // zero padding: no input there
                for (int kx = 0; kx < 3; ++kx) {
                    const int ix = x + kx - 1; if (ix < 0 || ix >= g) continue;
                    const float* w = S.w + (((size_t)c * 3 + ky) * 3 + kx) * S.cin;
                    double* d = &gi[((size_t)iy * g + ix) * S.cin];
                    for (int ci = 0; ci < S.cin; ++ci) d[ci] += v * (double)w[ci];
                }
            }
        }
        const int iy0 = std::max(cy0 - 1, 0), iy1 = std::min(cy1 + 1, g - 1), ix0 = std::max(cx0 - 1, 0), ix1 = std::min(cx1 + 1, g - 1);
        if (k == 0) { g_in0.swap(gi); return; }
        // back through the previous stage's pixel shuffle: ps[y*r+i][x*r+j][c] = conv[y][x][c*r*r + i*r + j]
        const fold_stage& P = st[k - 1];
        const int r = P.r, gp = grid[k - 1];
        gc.assign((size_t)gp * gp * P.cout, 0.0);
        for (int y = iy0; y <= iy1; ++y) for (int x = ix0; x <= ix1; ++x) for (int c = 0; c < S.cin; ++c) {
            const double v = gi[((size_t)y * g + x) * S.cin + c];
            if (v != 0.0) gc[((size_t)(y / r) * gp + x / r) * P.cout + c * r * r + (y % r) * r + (x % r)] = v;
        }
        cy0 = iy0 / r; cy1 = iy1 / r; cx0 = ix0 / r; cx1 = ix1 / r;
    }
}

// The stages' response to an all-zero input on the small image (the composite bias at every position).
void fold_bias(const std::vector<fold_stage>& st, const std::vector<int>& grid, std::vector<double>& out /*[g][g][cout_last]*/)
{
    std::vector<double> x((size_t)grid[0] * grid[0] * st[0].cin, 0.0);
    for (size_t k = 0; k < st.size(); ++k) {
        const fold_stage& S = st[k];
        const int g = grid[k];
        std::vector<double> yv((size_t)g * g * S.cout);
        for (int y = 0; y < g; ++y) for (int xx = 0; xx < g; ++xx) for (int c = 0; c < S.cout; ++c) {
            double acc = (double)S.b[c];
            for (int ky = 0; ky < 3; ++ky) {
                const int iy = y + ky - 1; if (iy < 0 || iy >= g) continue;
                for (int kx = 0; kx < 3; ++kx) {
                    const int ix = xx + kx - 1; if (ix < 0 || ix >= g) continue;
                    const float* w = S.w + (((size_t)c * 3 + ky) * 3 + kx) * S.cin;
                    const double* in = &x[((size_t)iy * g + ix) * S.cin];
                    for (int ci = 0; ci < S.cin; ++ci) acc += (double)w[ci] * in[ci];
                }
            }
            yv[((size_t)y * g + xx) * S.cout + c] = acc;
        }
        if (S.r == 1) { x.swap(yv); continue; }
        const int r = S.r, co = S.cout / (r * r);
        x.assign((size_t)g * r * g * r * co, 0.0);
        for (int y = 0; y < g; ++y) for (int xx = 0; xx < g; ++xx) for (int c = 0; c < co; ++c)
            for (int i = 0; i < r; ++i) for (int j = 0; j < r; ++j)
                x[((size_t)(y * r + i) * (g * r) + (xx * r + j)) * co + c] = yv[((size_t)y * g + xx) * S.cout + c * r * r + i * r + j];
    }
    out.swap(x);
}

uint16_t fold_bf16(double v)
{
    const float f = (float)v;
    uint32_t u; memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

}  // namespace

// Builds ctx->fold_w / fold_b for an EDSR-shaped net; a no-op for the other topologies.
// Layout: fold_w [class 9][chunk][tap 25][ks][lane 64][8] bf16 with row = lane % 32 of the chunk and
// ci = 16 ks + 8 (lane / 32) + e; fold_b [class][chunk][32] fp32.  In the place of the middle class, the main kernel's:
// [tap 25][kh][m][lane 64][8] with row = 16 m + lane % 16 and ci = 32 kh + 8 (lane / 16) + e; its biases by row.
rh_status rh_fold_weights(rh_ctx* ctx, const float* blob)
{
    const rh_net_desc& d = ctx->cfg.net;
    ctx->fold_chunks = 0;
    if (d.topology != RH_NET_EDSR || ctx->cfg.precision != RH_BF16) return RH_OK;
    const int C = d.channels, s = d.scale;
    if (C != 32 && C != 64) return RH_OK;
    const size_t nl = ctx->layers.size();
    std::vector<fold_stage> st;
    const int n_up = s == 4 ? 2 : 1;
    for (int u = 0; u < n_up; ++u) {
        const rh_layer& L = ctx->layers[nl - 1 - n_up + u];
        st.push_back({blob + L.w_off, blob + L.b_off, L.cin, L.cout, s == 4 ? 2 : s});
    }
    const rh_layer& T = ctx->layers[nl - 1];
    st.push_back({blob + T.w_off, blob + T.b_off, T.cin, T.cout, 1});
    std::vector<int> grid(st.size());
    grid[0] = 5;
    for (size_t k = 1; k < st.size(); ++k) grid[k] = grid[k - 1] * st[k - 1].r;
    const int gl = grid.back();                            // = 5 s
    const int R = 3 * s * s, n_chunks = s == 4 ? 2 : 1, ipc = s == 4 ? 2 : s, rows = 3 * s * ipc, KS = C / 16;
    std::vector<double> bias_all;
    fold_bias(st, grid, bias_all);
    // Wc[class][i][j][co][tap][ci]; the class's pixel sits at row / column 0, 2 or 4 of the 5 x 5 image
    std::vector<double> Wc((size_t)9 * R * 25 * C, 0.0);
    auto compose = [&](int job0, int job1) {
        std::vector<double> g;
        for (int job = job0; job < job1; ++job) {
            const int cls = job / R, o = job - cls * R, py = 2 * (cls / 3), px = 2 * (cls % 3);
            const int i = o / (3 * s), j = (o / 3) % s, co = o % 3;
            fold_gradient(st, grid, py * s + i, px * s + j, co, g);
            double* dst = &Wc[((size_t)cls * R + o) * 25 * C];
            for (int dy = -2; dy <= 2; ++dy) for (int dx = -2; dx <= 2; ++dx) {
                const int yy = py + dy, xx = px + dx;
                if (yy < 0 || yy >= 5 || xx < 0 || xx >= 5) continue;           // outside the image: t is zero there
                memcpy(dst + ((dy + 2) * 5 + (dx + 2)) * C, &g[((size_t)yy * 5 + xx) * C], sizeof(double) * C);
            }
        }
    };
    std::atomic<bool> out_of_memory{false};                // a thread that ended by an exception would end the process
    auto work = [&](int job0, int job1) { try { compose(job0, job1); } catch (const std::bad_alloc&) { out_of_memory = true; } };
    {
        const int jobs = 9 * R, nt = 8;
        std::vector<std::thread> th;
        th.reserve(nt);
        for (int t = 0; t < nt; ++t) {
            try { th.emplace_back(work, jobs * t / nt, jobs * (t + 1) / nt); }
            catch (const std::exception&) { work(jobs * t / nt, jobs * (t + 1) / nt); }      // no thread to be had
        }
        for (auto& t : th) t.join();
        if (out_of_memory) throw std::bad_alloc();
    }
    std::vector<uint16_t> wp((size_t)9 * n_chunks * 25 * KS * 64 * 8);
    std::vector<float> bp((size_t)9 * n_chunks * 32, 0.0f);
    size_t wi = 0;
    for (int cls = 0; cls < 9; ++cls)
        for (int m = 0; m < n_chunks; ++m) {
            const int py = 2 * (cls / 3), px = 2 * (cls % 3);
            if (cls == 4) {                                // the main kernel's, below
                wi += (size_t)25 * KS * 64 * 8;
                continue;
            }
            for (int tap = 0; tap < 25; ++tap)
                for (int ks = 0; ks < KS; ++ks)
                    for (int lane = 0; lane < 64; ++lane)
                        for (int e = 0; e < 8; ++e) {
                            const int rho = lane & 31, ci = ks * 16 + 8 * (lane >> 5) + e;
                            double v = 0.0;
                            if (rho < rows) {
                                const int il = rho / (3 * s), rem = rho - il * 3 * s, o = (m * ipc + il) * 3 * s + rem;
                                v = Wc[(((size_t)cls * R + o) * 25 + tap) * C + ci];
                            }
                            wp[wi++] = fold_bf16(v);
                        }
            for (int rho = 0; rho < rows; ++rho) {
                const int il = rho / (3 * s), rem = rho - il * 3 * s, i = m * ipc + il, j = rem / 3, co = rem % 3;
                bp[((size_t)cls * n_chunks + m) * 32 + rho] = (float)bias_all[((size_t)(py * s + i) * gl + (px * s + j)) * 3 + co];
            }
        }
    const int MT = (R + 15) / 16;
    wi = (size_t)4 * n_chunks * 25 * KS * 64 * 8;
    for (int tap = 0; tap < 25; ++tap)
        for (int kh = 0; kh < C / 32; ++kh)
            for (int m = 0; m < MT; ++m)
                for (int lane = 0; lane < 64; ++lane)
                    for (int e = 0; e < 8; ++e) {
                        const int o = 16 * m + (lane & 15), ci = kh * 32 + 8 * (lane >> 4) + e;
                        wp[wi++] = fold_bf16(o < R ? Wc[(((size_t)4 * R + o) * 25 + tap) * C + ci] : 0.0);
                    }
    for (int o = 0; o < R; ++o) {
        const int i = o / (3 * s), j = o / 3 % s, co = o % 3;
        bp[(size_t)4 * n_chunks * 32 + o] = (float)bias_all[((size_t)(2 * s + i) * gl + (2 * s + j)) * 3 + co];
    }
    RH_HIP(ctx, hipMalloc(&ctx->fold_w, wp.size() * 2));
    RH_HIP(ctx, hipMalloc((void**)&ctx->fold_b, bp.size() * 4));
    RH_HIP(ctx, hipMemcpy(ctx->fold_w, wp.data(), wp.size() * 2, hipMemcpyHostToDevice));
    RH_HIP(ctx, hipMemcpy(ctx->fold_b, bp.data(), bp.size() * 4, hipMemcpyHostToDevice));
    ctx->fold_chunks = n_chunks;
    return RH_OK;
}

template <int CIN, int S, bool LIST>
static hipError_t launch_fold(rh_ctx* ctx, const fold_args& a)
{
    using L = fold_shape<CIN, S>;
    static bool attr_done[RH_MAX_DEVICES] = {};
    if (!attr_done[ctx->device]) {
        hipError_t e = hipFuncSetAttribute((const void*)k_conv_fold<CIN, S, LIST>, hipFuncAttributeMaxDynamicSharedMemorySize, L::LDS);
        if (e != hipSuccess) return e;
        attr_done[ctx->device] = true;
    }
    hipLaunchKernelGGL((k_conv_fold<CIN, S, LIST>), dim3(ctx->n_cu), dim3(L::WAVES * 64), L::LDS, ctx->stream, a);
    return hipGetLastError();
}

template <int CIN, bool LIST>
static hipError_t launch_fold(rh_ctx* ctx, const fold_args& a)
{
    const int s = ctx->cfg.net.scale;
    return s == 4 ? launch_fold<CIN, 4, LIST>(ctx, a) : s == 3 ? launch_fold<CIN, 3, LIST>(ctx, a) : launch_fold<CIN, 2, LIST>(ctx, a);
}

// t: the body's output [N][H][W][C] bf16 -> raw network output fp32 [N][sH][sW][3]; one launch.
rh_status rh_launch_fold(rh_ctx* ctx, const __bf16* t, float* out, int N, int H, int W, const uint32_t* n_valid, int rev,
                         const uint32_t* tile_list, const uint32_t* n_list)
{
    fold_args a;
    a.tile_list = tile_list; a.n_list = n_list;
    a.in = t; a.wp = (const uint4*)ctx->fold_w; a.bias = ctx->fold_b; a.out = out; a.n_valid = n_valid;
    a.N = N; a.H = H; a.W = W; a.n_chunks = ctx->fold_chunks; a.rev = rev;
    // Needed-region mode: a pasted macroblock lies at least `halo` pixels inside its box, hence inside
    // the bin, so with a halo no pasted pixel is on the outermost ring.
    a.ring = !(tile_list && ctx->cfg.halo >= 1);
    // lists of tiles come from the needed-region mode, which takes nets of 64 channels only (rh_enhance_needed)
    if (ctx->cfg.net.channels == 64) RH_HIP(ctx, (tile_list ? launch_fold<64, true>(ctx, a) : launch_fold<64, false>(ctx, a)));
    else if (tile_list) RH_FAIL(ctx, RH_E_UNIMPLEMENTED, "a list of tiles with %d channels", ctx->cfg.net.channels);
    else RH_HIP(ctx, (launch_fold<32, false>(ctx, a)));
    return RH_OK;
}
