// Two 3x3 convs of a 64-channel net in one launch: a residual block (out = x + conv2(relu(conv1(x)))), or two ReLU layers.
//
// The tensor between the two convs and the skip values stay in LDS: a launch reads x and writes out, where a launch per conv
// (conv_mfma_duo.hip) moves two and a half times as much.  It is computed as a stream of rows.  A workgroup takes a run of rows of a
// strip of columns, top to bottom; an input row is read from memory once and feeds the sums of three rows of the tensor between,
// a finished row of which feeds three output rows: no patch, nothing of a row is computed twice, and a strip as wide as the
// image (up to 128 pixels) has no columns beside it to compute twice either.
//
// Waves 0-3 are conv1, waves 4-7 conv2: a wave has 16 output channels of all pixels of the strip, its conv's 18 weight fragments in
// registers, and the sums of three rows.  Each SIMD holds one wave of each.  In iteration t
//   conv1 makes the products of the stream's input row t, which finish the row above it of the tensor between: ReLU, rounding, to LDS; and stores
//         the output row that conv2 rounded in iteration t - 1;
//   conv2 copies input row t + 1 to LDS; rounds the output row that its last products finished, + x, rounding, into x's place in LDS; and makes the
//         products of the row that conv1 finished in iteration t - 1, which finish the output row above that one;
// and all meet at one barrier.  conv1's products come first, conv2's rounding beside them, then conv2's products beside what conv1 has left to do.
// LDS, rows of 16 NT + 8 pixels of 128 bytes, 16-byte channel groups swizzled by the pixel: 7 input rows (row t, copied in in t - 1, is x's place for
// what conv2 finishes in iteration t + 3, rounds in t + 4 and conv1 stores in t + 5), 2 rows of the tensor between.
//
// A run that begins inside an image works on two rows more above it and two below.  Sums start from the bias as the first product's C operand and
// run over (ky, kx, half of K), as in the other kernels of the body: the same bits.
//
// What bounds it: the chip's power limit, and the instructions beside the products - a product of 16 cycles hides two of them, of
// both waves together.  EDSR x4, us, a launch per conv / this: 55 bins of 128 x 128 2 156 / 1 958, 76: 2 946 / 2 630, 150: 5 813 / 4 961; with images and
// weights of zeros 1 675 / 1 522, 2 375 / 1 990, 4 830 / 3 640.  An iteration of 8 tiles takes 5 900 cycles, of which 4 608 are products.  With the
// rounding of a tile between the products of the next one it took 6 600, with conv2's rounding and stores all ahead of its products 6 500.
#include "conv_mfma64.h"

#define B64_RING 7

// The sums live in registers that this file names itself: left to the compiler, which would give a row's sums other registers where they
// are finished, they are copied in every turn of the loop and do not fit.  From B64_X on: the row that is finished next, then the one after it, then
// the newest, 4 NT each, then the bias.  Every statement that names one lists all of them as overwritten, so that nothing of the compiler's that lives
// across such a statement lies there.  What lives between two of them only, it could still put there: the build reads the code that the compiler made
// of this file and fails where it has (build.py, named_registers).
#define B64_X 156
#define B64_REGS "v156", "v157", "v158", "v159", "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167", "v168", "v169", "v170", "v171", "v172", "v173", \
    "v174", "v175", "v176", "v177", "v178", "v179", "v180", "v181", "v182", "v183", "v184", "v185", "v186", "v187", "v188", "v189", "v190", "v191", \
    "v192", "v193", "v194", "v195", "v196", "v197", "v198", "v199", "v200", "v201", "v202", "v203", "v204", "v205", "v206", "v207", "v208", "v209", \
    "v210", "v211", "v212", "v213", "v214", "v215", "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", "v224", "v225", "v226", "v227", \
    "v228", "v229", "v230", "v231", "v232", "v233", "v234", "v235", "v236", "v237", "v238", "v239", "v240", "v241", "v242", "v243", "v244", "v245", \
    "v246", "v247", "v248", "v249", "v250", "v251", "v252", "v253", "v254", "v255"
template <int D, int C>
__device__ __forceinline__ void b64_mfma(const bf16x8& x, const bf16x8& y)       // v[D..D+3] = v[C..C+3] + x y
{
    asm volatile("v_mfma_f32_16x16x32_bf16 v[%c0:%c1], %2, %3, v[%c4:%c5]" :: "n"(D), "n"(D + 3), "v"(x), "v"(y), "n"(C), "n"(C + 3) : B64_REGS);
}
template <int D, int C, int D2, int C2>
__device__ __forceinline__ void b64_mfma2(const bf16x8& x, const bf16x8& x2, const bf16x8& y)      // two with the same y
{
    asm volatile("v_mfma_f32_16x16x32_bf16 v[%c0:%c1], %2, %3, v[%c4:%c5]\n\tv_mfma_f32_16x16x32_bf16 v[%c6:%c7], %8, %3, v[%c9:%c10]"
                 :: "n"(D), "n"(D + 3), "v"(x), "v"(y), "n"(C), "n"(C + 3), "n"(D2), "n"(D2 + 3), "v"(x2), "n"(C2), "n"(C2 + 3) : B64_REGS);
}
template <int I>
__device__ __forceinline__ uint2 b64_round()                 // v[I..I+3] as four bf16
{
    uint2 p;
    asm volatile("v_cvt_pk_bf16_f32 %0, v%c1, v%c2" : "=v"(p.x) : "n"(I), "n"(I + 1) : B64_REGS);
    asm volatile("v_cvt_pk_bf16_f32 %0, v%c1, v%c2" : "=v"(p.y) : "n"(I + 2), "n"(I + 3) : B64_REGS);
    return p;
}
// before a vector instruction reads sums
__device__ __forceinline__ void b64_settle() { asm volatile("s_nop 15\n\ts_nop 3" ::: "memory"); }

struct block64_args {
    const __bf16* in; __bf16* out;
    const uint4 *w1, *w2;
    const float *b1, *b2;
    const uint32_t* n_valid;
    int N, H, W;
    int strips, wo;          // strips of an image, columns of all but the last
};

// Row of a stream: input row r of strip `strip` of image n, whose output rows [y0, y1) the run has.  n < 0: there is none.
struct block64_row { int n, strip, y0, y1, r; };

template <int NT, int NT2, bool RES>
__global__ __launch_bounds__(512) void k_conv_mfma_block64(block64_args a)
{
    constexpr int PIXB = 128, ROWPX = 16 * NT + 8, ROWB = ROWPX * PIXB;
    constexpr int X = B64_X, Y = X + 4 * NT, Z = Y + 4 * NT, BIAS = Z + 4 * NT;
    static_assert(BIAS + 4 <= 256, "registers kept");
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    uint8_t* lds_m = lds + B64_RING * ROWB;
    const int tid = threadIdx.x, lane = tid & 63;
    const int conv2 = __builtin_amdgcn_readfirstlane(tid >> 8), m = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);

    const int n_img = a.n_valid ? min((int)*a.n_valid, a.N) : a.N;
    const int G = gridDim.x, wg = (G % 8 == 0) ? (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8 : blockIdx.x;
    const int total = max(n_img, 0) * a.strips * a.H, share = total / G, more = total - share * G;
    int pos = wg * share + min(wg, more);
    const int end = pos + share + (wg < more);
    if (pos >= end) return;

    bf16x8 A[3][6];
    {
        const uint4* w = (conv2 ? a.w2 : a.w1) + m * 64 + lane;
#pragma unroll
        for (int ky = 0; ky < 3; ++ky)
#pragma unroll
            for (int f = 0; f < 6; ++f) A[ky][f] = *(const bf16x8*)(w + (ky * 6 + f) * 256);
    }
    {
        const float4 v = *(const float4*)((conv2 ? a.b2 : a.b1) + m * 16 + (lane >> 4) * 4);
        asm volatile("v_mov_b32 v%c0, %4\n\tv_mov_b32 v%c1, %5\n\tv_mov_b32 v%c2, %6\n\tv_mov_b32 v%c3, %7"
                     :: "n"(BIAS), "n"(BIAS + 1), "n"(BIAS + 2), "n"(BIAS + 3), "v"(v.x), "v"(v.y), "v"(v.z), "v"(v.w) : B64_REGS);
    }
    const uint32_t img_bytes = (uint32_t)a.H * a.W * PIXB;
    const size_t img_elems = (size_t)a.H * a.W * 64;

    auto piece = [&](block64_row& c) __attribute__((always_inline)) {
        if (pos >= end) { c.n = -1; return; }
        const int col = pos / a.H;
        c.y0 = pos - col * a.H; c.y1 = min(a.H, c.y0 + end - pos);
        c.n = col / a.strips; c.strip = col - c.n * a.strips;
        c.r = max(c.y0 - 2, -1);
        pos += c.y1 - c.y0;
    };
    auto next = [&](block64_row& c) __attribute__((always_inline)) {
        if (c.n < 0) return;
        if (++c.r > min(c.y1, a.H - 1) + 1) piece(c);
    };
    auto inside = [&](const block64_row& c) __attribute__((always_inline)) { return c.n >= 0 && (uint32_t)c.r < (uint32_t)a.H; };
    auto left = [&](int strip) __attribute__((always_inline)) { return strip > 0 ? 1 : 0; };   // columns of the tensor between that lie left of the strip
    auto wrap = [&](int slot) __attribute__((always_inline)) { return slot >= B64_RING ? slot - B64_RING : slot; };
    // `lane` passes through an empty asm statement wherever addresses are made of it: kept over the loop they would not fit the registers
    auto lane_now = [&]() __attribute__((always_inline)) { int l = lane; asm volatile("" : "+v"(l)); return l; };

    // Fragment i of a row: (kx, half of K) = i / T of tile i % T of T, NT for conv1 and NT2 for conv2.  Two at a time, so that they take one wait; read two pairs ahead.
    bf16x8 B[6];
    uint32_t b_lane[3];
    {
        const int l = lane_now();
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) b_lane[kx] = (uint32_t)(((l & 15) + kx) * PIXB + (((l >> 4) ^ (((l & 15) + kx) & 7)) << 4));
    }
    auto load = [&](const uint8_t* row, int i, int T) __attribute__((always_inline)) {
        const int f = i / T, n = i % T;
        B[i % 6] = *(const bf16x8*)(row + (b_lane[f >> 1] ^ ((f & 1) << 6)) + n * (16 * PIXB));
    };
    auto load_first = [&](const uint8_t* row, int T) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) load(row, i, T);
        __builtin_amdgcn_sched_barrier(0);
    };
    // The products of a row whose first fragments are there.  At most two other instructions hide behind a product.
    auto products = [&](const uint8_t* row, auto t_c) __attribute__((always_inline)) {
        constexpr int T = decltype(t_c)::value;
        auto frag = [&](auto i_c) __attribute__((always_inline)) {
            constexpr int i = decltype(i_c)::value, f = i / T, n = i % T, x = X + 4 * n, y = Y + 4 * n, z = Z + 4 * n;
            const bf16x8 &a0 = A[0][f], &a1 = A[1][f], &a2 = A[2][f], &b = B[i % 6], &c = B[(i + 1) % 6];
            if constexpr (i % 2 == 0) asm volatile("" :: "v"(b), "v"(c));
            // There and back over the three rows of taps: from one product to the next only one operand changes, which takes less power (from
            // registers 1.97 PFLOP/s with the rows always in the same order, 2.03 with this).  f = 0: the sums move on by a row, the oldest first.
            constexpr bool back = f && i % 2;
            if constexpr (back) b64_mfma<z, z>(a0, b); else b64_mfma<x, f ? x : y>(a2, b);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i + 4 < 6 * T) load(row, i + 4, T);   // in the place of a fragment of the pair before this one
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (back) b64_mfma2<y, y, x, x>(a1, a2, b); else b64_mfma2<y, f ? y : z, z, f ? z : BIAS>(a1, a0, b);
            __builtin_amdgcn_sched_barrier(0);
        };
        conv64_each<6 * T>(frag);
    };
    // A row of zeros: the sums move on.
    auto zeros = [&]() __attribute__((always_inline)) {
        bf16x8 none = {};
        asm volatile("" : "+v"(none));
        b64_settle();
        auto tile = [&](auto n_c) __attribute__((always_inline)) {
            constexpr int n = decltype(n_c)::value, x = X + 4 * n, y = Y + 4 * n, z = Z + 4 * n;
            const bf16x8& o = none;
            b64_mfma<x, y>(o, o);
            b64_mfma<y, z>(o, o);
            b64_mfma<z, BIAS>(o, o);
        };
        conv64_each<NT>(tile);
    };
    // copies input row c.r to its place; wave m the pieces m, m + 4, ... of 8 pixels
    auto copy_row = [&](const block64_row& c, int slot) __attribute__((always_inline)) {
        if (!inside(c)) return;
        __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc((void*)(a.in + (size_t)c.n * img_elems), 0, img_bytes, RSRC_FLAGS);
        const int x0 = c.strip * a.wo - left(c.strip) - 1;   // column of the place's first pixel
        const int l = lane_now(), px = m * 8 + (l >> 3), gx = x0 + px;
        const uint32_t off = (uint32_t)((c.r * a.W + gx) * PIXB + (((l & 7) ^ (l >> 3)) << 4));
#pragma unroll
        for (int i = 0; i < (ROWPX / 8 + 3) / 4; ++i) {
            if (i * 4 + m >= ROWPX / 8) break;
            // inline asm, with no register written: behind the builtin the compiler has every LDS read wait for the copy
            const uint32_t to = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)(lds + slot * ROWB + (i * 4 + m) * 1024));
            const uint32_t o = (uint32_t)(gx + i * 32) < (uint32_t)a.W ? off + i * (32 * PIXB) : OOB_OFF;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" :: "s"(to), "v"(o), "s"(rin) : "memory", "m0");
        }
    };

    block64_row before, c;                                   // rows t - 1 and t of the stream
    piece(c);
    before.n = -1;
    if (conv2) copy_row(c, 0);
    lds_dma_wait();
    lds_barrier();
    // the output row that was finished last, the one that was rounded last, one that waits for the row of zeros below the image; n < 0: none
    struct out_row { int n, strip, y; };
    out_row done = {-1, 0, 0}, rounded = {-1, 0, 0}, last = {-1, 0, 0};
    // What conv2 does in this iteration, with row before.r - 1 of the tensor between: its products finish the output row above it
    enum { NOTHING, PRODUCTS, ZEROS };
    auto turn = [&]() __attribute__((always_inline)) {
        const int q = before.r - 1;
        rounded = done;
        done.n = -1;
        if (before.n >= 0 && q >= max(before.y0 - 1, 0)) {
            if (q > before.y0) done = {before.n, before.strip, q - 1};
            if (q == a.H - 1 && before.y1 == a.H) last = {before.n, before.strip, q};
            return PRODUCTS;
        }
        if (last.n >= 0) { done = last; last.n = -1; return ZEROS; }
        return before.n >= 0 && q == -1 ? ZEROS : NOTHING;
    };
    int slot = 0, par = 0;
    // iterations: all rows of the stream, and the four that conv2, its rounding and the stores are behind
    if (!conv2) {
        for (int behind = 0; behind < 4;) {
            if (c.n >= 0) {                                  // row r - 1 of the tensor between; columns outside the image are zero
                __builtin_amdgcn_s_setprio(2);
                if (inside(c)) {
                    load_first(lds + slot * ROWB, NT);
                    products(lds + slot * ROWB, std::integral_constant<int, NT>{});
                } else zeros();
                __builtin_amdgcn_s_setprio(0);
                b64_settle();
                const int l = lane_now();
                uint8_t* mid = lds_m + par * ROWB;
                const int xs = c.strip * a.wo - left(c.strip), shift = 1 - left(c.strip), px = (l & 15) + shift, room = a.W - xs - (l & 15);
                uint8_t* to = mid + px * PIXB + (((m * 2 + (l >> 5)) ^ (px & 7)) << 4) + (l >> 4 & 1) * 8;
                auto write = [&](auto edge_c) __attribute__((always_inline)) {
                    auto tile = [&](auto n_c) __attribute__((always_inline)) {
                        constexpr int n = decltype(n_c)::value;
                        uint2 pk = b64_round<X + 4 * n>();
                        pk.x = relu_bf16x2(pk.x); pk.y = relu_bf16x2(pk.y);
                        if constexpr (decltype(edge_c)::value) { const bool in = n * 16 < room; pk.x = in ? pk.x : 0u; pk.y = in ? pk.y : 0u; }
                        *(uint2*)(to + n * (16 * PIXB)) = pk;
                    };
                    conv64_each<NT>(tile);
                };
                if (xs + 16 * NT > a.W) write(std::integral_constant<bool, true>{}); else write(std::integral_constant<bool, false>{});
                // the columns beside the image that no product's lane has: lanes 0-3 the left one, 4-7 the right one
                const int right = a.W - c.strip * a.wo + 1, side = (l & 4) ? right : 0;
                if (l < 8 && ((l & 4) ? right >= 16 * NT + shift && right < ROWPX : shift == 1))
                    *(uint2*)(mid + side * PIXB + (((m * 2 + (l >> 1 & 1)) ^ (side & 7)) << 4) + (l & 1) * 8) = make_uint2(0, 0);
            }
            if (rounded.n >= 0) {                            // by conv2 in the last iteration
                __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc((void*)(a.out + (size_t)rounded.n * img_elems), 0, img_bytes, RSRC_FLAGS);
                const int xo = rounded.strip * a.wo, w = min(a.wo, a.W - xo);
                const int l = lane_now(), j = m * 8 + (l >> 3), ci = j + left(rounded.strip) + 1;
                const uint32_t off = (uint32_t)((rounded.y * a.W + xo + j) * PIXB + ((l & 7) << 4));
                const uint8_t* at = lds + wrap(slot + 2) * ROWB + ci * PIXB + (((l & 7) ^ (ci & 7)) << 4);       // slot - 5
                uint4 v[(NT + 1) / 2];
#pragma unroll
                for (int i = 0; i < (NT + 1) / 2; ++i) v[i] = *(const uint4*)(at + i * (32 * PIXB));
#pragma unroll
                for (int i = 0; i < (NT + 1) / 2; ++i) {
                    const i32x4 o = {(int)v[i].x, (int)v[i].y, (int)v[i].z, (int)v[i].w};
                    __builtin_amdgcn_raw_buffer_store_b128(o, rout, j + i * 32 < w ? off + i * (32 * PIXB) : OOB_OFF, 0, ST_THROUGH);
                }
            }
            if (c.n < 0) ++behind;
            turn();
            before = c; next(c);
            slot = wrap(slot + 1); par ^= 1;
            lds_barrier();
        }
        return;
    }
    for (int behind = 0; behind < 4;) {
        const uint8_t* row = lds_m + (par ^ 1) * ROWB;
        load_first(row, NT2);                                // of no use where there are no products
        block64_row ahead = c;
        next(ahead);
        copy_row(ahead, wrap(slot + 1));
        if (done.n >= 0) {                                   // rounding, + x, rounding, into x's place.  (No b64_settle(), which would cost 0.3 %: the last product lies
                                                             // a barrier, the fragments' loads and a copy back, 47 wait states at least; the build checks for 20.)
            const int l = lane_now(), ci = (l & 15) + left(done.strip) + 1;
            uint8_t* at = lds + wrap(slot + 3) * ROWB + ci * PIXB + (((m * 2 + (l >> 5)) ^ (ci & 7)) << 4) + (l >> 4 & 1) * 8;       // slot - 4
            uint2 x[RES ? NT2 : 1];
            if constexpr (RES)
#pragma unroll
                for (int n = 0; n < NT2; ++n) x[n] = *(const uint2*)(at + n * (16 * PIXB));
            auto tile = [&](auto n_c) __attribute__((always_inline)) {
                constexpr int n = decltype(n_c)::value;
                uint2 pk = b64_round<X + 4 * n>();
                if constexpr (RES) {
                    pk.x = pack_bf16x2(bf16_lo(pk.x) + bf16_lo(x[n].x), bf16_hi(pk.x) + bf16_hi(x[n].x));
                    pk.y = pack_bf16x2(bf16_lo(pk.y) + bf16_lo(x[n].y), bf16_hi(pk.y) + bf16_hi(x[n].y));
                } else { pk.x = relu_bf16x2(pk.x); pk.y = relu_bf16x2(pk.y); }
                *(uint2*)(at + n * (16 * PIXB)) = pk;
            };
            conv64_each<NT2>(tile);
        }
        const int what = turn();
        __builtin_amdgcn_s_setprio(1);
        if (what == PRODUCTS) products(row, std::integral_constant<int, NT2>{}); else if (what == ZEROS) zeros();
        __builtin_amdgcn_s_setprio(0);
        if (c.n < 0) ++behind;
        before = c; c = ahead;
        slot = wrap(slot + 1); par ^= 1;
        lds_dma_wait();
        lds_barrier();
    }
}

template <int NT, int NT2, bool RES>
static hipError_t launch_block64(hipStream_t stream, int device, int grid, const block64_args& a)
{
    constexpr int lds = (B64_RING + 2) * (16 * NT + 8) * 128;
    static bool attr_done[RH_MAX_DEVICES] = {};            // the attribute is per device
    if (!attr_done[device]) {
        hipError_t e = hipFuncSetAttribute((const void*)k_conv_mfma_block64<NT, NT2, RES>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_done[device] = true;
    }
    hipLaunchKernelGGL((k_conv_mfma_block64<NT, NT2, RES>), dim3(grid), dim3(512), lds, stream, a);
    return hipGetLastError();
}

// Strips of equal width, as few 16-pixel tiles in all (of conv1, `tiles` a strip, and of conv2, `tiles2`) as can be had with 4 to 8 a strip.
// false: none fit.
bool rh_block64_strips(int W, int* strips, int* wo, int* tiles, int* tiles2)
{
    int best = 0;
    for (int n = 1; n <= (W + 47) / 48; ++n) {
        const int w = (W + n - 1) / n, t = (w + (n > 1) + (n > 2) + 15) / 16, t2 = (w + 15) / 16;
        if (t < 4 || t > 8 || (n - 1) * w >= W) continue;
        if (!best || n * (t + t2) < best) { best = n * (t + t2); *strips = n; *wo = w; *tiles = t; *tiles2 = t2; }
    }
    return best > 0;
}

hipError_t rh_launch_block64(rh_ctx* ctx, const rh_layer& L1, const rh_layer& L2, const __bf16* in, __bf16* out, int N, int H, int W,
                             bool res, const uint32_t* n_valid)
{
    block64_args a;
    a.in = in; a.out = out; a.n_valid = n_valid; a.N = N; a.H = H; a.W = W;
    a.w1 = (const uint4*)((const uint8_t*)ctx->wpack + L1.wp_off); a.w2 = (const uint4*)((const uint8_t*)ctx->wpack + L2.wp_off);
    a.b1 = ctx->bpack + L1.bp_off; a.b2 = ctx->bpack + L2.bp_off;
    int t, t2;
    if (!rh_block64_strips(W, &a.strips, &a.wo, &t, &t2)) return hipErrorInvalidValue;
#define B64(NT, NT2) if (t == NT && t2 == NT2) return res ? launch_block64<NT, NT2, true>(ctx->stream, ctx->device, ctx->n_cu, a) : launch_block64<NT, NT2, false>(ctx->stream, ctx->device, ctx->n_cu, a)
    B64(4, 3); B64(4, 4); B64(5, 4); B64(5, 5); B64(6, 5); B64(6, 6); B64(7, 6); B64(7, 7); B64(8, 7); B64(8, 8);
#undef B64
    return hipErrorInvalidValue;
}
