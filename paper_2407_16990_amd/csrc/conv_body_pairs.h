// A few images in k_conv_mfma_body (conv_body.hip): two layers a unit.
//
// With a unit a workgroup and layer, a layer of the body is a chain: words looked at, patch, 2 us of products, rounding, stores, words; 7.9 us.
// Here a unit is TH rows of 30 pixels of TWO layers - a residual block, or two ReLU layers -, so that half of the chain's links fall
// away, for products of TH + 2 rows of 32 pixels in the first of them.  All eight waves compute both layers: a wave has 32 of the 64 channels of
// every fourth run of 16 pixels.
//   LDS: two or three thirds (ky) of a layer's weights, and the patch, TH + 4 rows of 34 pixels, whose place the tensor between the layers takes.  A third
//   that all waves are through with is loaded over by one that is used later.
//   A workgroup has one unit, the same in every step of two layers: what it makes stays in its patch, and only the two rows and columns around
//   it come from its neighbours through memory.  (Where workgroups came too late for the roll, a workgroup has more than one unit: whole patches.)
//   Steps write to `a` and `t` in turn.  A unit's word says how many steps it has done; a step starts when the 3 x 3 around say so.  Whoever
//   read the old values of what it writes lies among the same 3 x 3, and had read them before its word.
// A unit's word has a 128-byte line of its own.  Side by side, 240 words in 8 lines that 1920 waves look at, a step of 3 bins took 27 600 cycles, and
// 22 200 so; with a word a wave, 8 in a line, 24 000.
// TH is the least of 4, 6, .. 22 with which there is a workgroup for every unit; where 22 rows are not enough, the batch goes a layer at a time, as it
// does with 2 units a workgroup of fewer rows.  us, EDSR x4 on 128 x 128 bins, a layer / two layers a unit: 1 bin 248 / 136, 2: 261 / 159, 3: 272 / 189, 4: 286 / 228,
// 6: 328 / 285, 7: 347 / 339, 8: 385 / 364; 12 of 96 x 96 335 / 334; 5 of 160 x 160 383 / 342; a frame of 480 x 272 399 / 324.
// What bounds it: of a step's 22 200 cycles on 3 bins 10 400 are products, 3 000 the wait for words and what lies around, 2 200 stores until they are
// acknowledged; from 4 bins on also the instructions of the two roundings, and the slower of the two waves of a SIMD.
// Sums as in the other kernels of the body (conv_mfma64.h): the same bits.
#pragma once
#include "conv_mfma64.h"

#define BODY_PAIR_MOST 22
#define BODY_PAIR_COLS 30                // output columns of a unit: the 32 of the tensor between, less one at each side

// Rows of a unit, 0: a layer at a time.  There are at most `grid` units, of which each has BODY_PAIR_WORDS words of `done`.
__host__ __device__ __forceinline__ long long body_pair_units(int images, int H, int W, int rows)
{
    return (long long)images * ((H + rows - 1) / rows) * ((W + BODY_PAIR_COLS - 1) / BODY_PAIR_COLS);
}
__host__ __device__ __forceinline__ int body_pair_rows(int images, int H, int W, int grid)
{
    for (int rows = 4; rows <= BODY_PAIR_MOST; rows += 2)
        if (body_pair_units(images, H, W, rows) <= grid) return rows;
    return 0;
}
#define BODY_PAIR_THIRD (3 * 64 * 64 * 2)
#define BODY_PAIR_SLOTS(rows) ((rows) > 16 ? 2 : 3)                         // thirds of a layer's weights in LDS
#define BODY_PAIR_LDS(rows) (BODY_PAIR_SLOTS(rows) * BODY_PAIR_THIRD + ((rows) + 4) * PW * 128 + 512)

// a and b hold channels 4 g + {0..3} of tile 0 and of tile 1 in the lanes of row g; after this the lane of row g has channels
// 8 (g / 2) + {0..7} of tile g % 2
__device__ __forceinline__ uint4 body_pair_lanes(uint2 a, uint2 b)
{
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    const u32x2 x = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false), y = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
    return make_uint4(x[0], y[0], x[1], y[1]);
}

// wt[k]: third k (ky) of the weights.  A fragment of the weights is read a sub-step ahead, one of the patch R - 1 products' pairs ahead.
template <int N, typename H>
__device__ __forceinline__ void body_pair_products(f32x4 (&acc)[N][2], const f32x4 (&bias)[2], const uint8_t* const (&wt)[3], const uint8_t* rows, int lane, int shift, H& hook)
{
    constexpr int R = 8;
    bf16x8 A[2][2], B[R];
    const int px0 = (lane & 15) + shift, grp = lane >> 4;
    auto load_a = [&](int st, int m) __attribute__((always_inline)) { A[st & 1][m] = *(const bf16x8*)(wt[st / 6] + ((st % 6 * 4 + m) << 10)); };
    auto load_b = [&](int g) __attribute__((always_inline)) {              // run g % N of sub-step g / N
        const int st = g / N, j = g % N, ky = st / 6, px = px0 + st / 2 % 3;
        B[g % R] = *(const bf16x8*)(rows + px * 128 + (((grp ^ (px & 7)) << 4) ^ ((st & 1) << 6)) + (2 * j + ky) * (PW * 128));
    };
    load_a(0, 0); load_a(0, 1);
#pragma unroll
    for (int g = 0; g < R - 1; ++g) load_b(g);
    auto sub = [&](auto st_c) __attribute__((always_inline)) {
        constexpr int st = decltype(st_c)::value;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if (j < 2 && st + 1 < C64_SUBSTEPS) load_a(st + 1, j);
            if (st * N + j + R - 1 < C64_SUBSTEPS * N) load_b(st * N + j + R - 1);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int m = k ^ (j & 1);
                acc[j][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A[st & 1][m], B[(st * N + j) % R], st == 0 ? bias[m] : acc[j][m], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        hook(st_c);
    };
    conv64_each<C64_SUBSTEPS>(sub);
}

// k_conv_mfma_body's arguments, read anew for each of its ways: what is worked out of them for one is not kept in registers for another
__device__ __forceinline__ body_args body_args_anew(int& n_img, int& wg, int& G)
{
    auto args = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args), "+s"(n_img), "+s"(wg), "+s"(G));
    return *(const body_args*)args;
}

// lds: BODY_PAIR_LDS(TH) bytes; stored: a zeroed word of LDS, as is lost (1: a wave has given up a wait).  All waves of workgroup wg of the G.
template <int TH, bool KEEP>
__device__ __forceinline__ void body_pairs(uint8_t* lds, uint32_t* stored, uint32_t* s_lost, int n_img, int wg, int G)
{
    const body_args a = body_args_anew(n_img, wg, G);
    constexpr int PIXB = 128, THIRD = BODY_PAIR_THIRD, WBYTES = 3 * THIRD, SLOTS = BODY_PAIR_SLOTS(TH), N1 = (TH + 2) / 2, N2 = TH / 2;
    constexpr int NP = ((TH + 4) * PW * 8 + 63) / 64, NPW = (NP + 7) / 8;   // loads of 64 x 16 bytes of a patch, of a wave
    constexpr int NH = (4 * PW + 4 * TH) * 8, NHW = (NH + 511) / 512;       // 16-byte pieces around a unit, of a thread
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int mh = wave & 1, hf = wave >> 1 & 1, rp = wave >> 2;            // channels 32 mh + .., columns 16 hf + .., rows 2 i + rp
    uint8_t* lds_p = lds + SLOTS * THIRD;
    const uint8_t* rows = lds_p + rp * (PW * PIXB) + hf * (16 * PIXB);
    // What is worked out of the lane is worked out anew in every phase (it passes through an empty asm statement): kept over the loop it would not
    // fit the registers.  Pixel and 16-byte group of a lane's 8 channels (body_pair_lanes):
    auto lane_now = [&]() __attribute__((always_inline)) { int l = lane; if (TH > 14) asm volatile("" : "+v"(l)); return l; };
    auto col_of = [&](int l) __attribute__((always_inline)) { return hf * 16 + (l & 15); };
    auto grp_of = [&](int l) __attribute__((always_inline)) { return mh * 4 + (l >> 4 & 1) * 2 + (l >> 5); };

    const int cells_x = (a.W + BODY_PAIR_COLS - 1) / BODY_PAIR_COLS, cells_y = (a.H + TH - 1) / TH, cells_img = cells_x * cells_y, units = n_img * cells_img;
    const uint32_t img_bytes = (uint32_t)a.H * a.W * PIXB;
    const size_t img_elems = (size_t)a.H * a.W * 64;
    const int steps = (a.layers + 1) / 2;
    const bool stay = G >= units;                            // a workgroup has the same unit in every step: what it makes stays in the patch
    __bf16* const out_last = a.topology == RH_NET_EDSR || (a.topology == RH_NET_PLAIN && !(a.layers & 1)) ? a.t : a.a;      // where the body's output is
    __bf16* const out_other = out_last == a.t ? a.a : a.t;
    auto out_of = [&](int s) __attribute__((always_inline)) { return (steps - 1 - s) & 1 ? out_other : out_last; };
    __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)a.wp, 0, (uint32_t)a.layers * WBYTES, RSRC_FLAGS);
    // 1 KB to `at` behind the workgroup's LDS + 1024 wave.  No register is written: no wait of the compiler's
    const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(const __attribute__((address_space(3))) uint8_t*)lds + wave * 1024);
    const uint32_t wlane_off = wave * 1024 + lane * 16;
    auto barrier = [&]() __attribute__((always_inline)) { lds_barrier(); __builtin_amdgcn_sched_barrier(0); };
    // The thirds of all layers' weights are used in turn, number t in slot t % SLOTS: loaded there when all waves have read number t - SLOTS
    auto load_third = [&](int layer, int k, int slot) __attribute__((always_inline)) {       // of the last layer where there is none: not used
        const uint32_t from = (uint32_t)min(layer, a.layers - 1) * WBYTES + k * THIRD;
#pragma unroll
        for (int i = 0; i < THIRD / 8192; ++i)
            asm volatile("s_add_u32 m0, %0, %c1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, %4 offen lds"
                         :: "s"(base + slot * THIRD), "n"(i * 8192), "v"(wlane_off), "s"(rw), "s"(from + i * 8192) : "memory", "scc", "m0");
    };
    int par = 0;                                             // two slots: that of the layer's first third
    auto slot_of = [&](int k) __attribute__((always_inline)) { return SLOTS == 3 ? k : (k + par) & 1; };
    // Between two sub-steps of a layer; its next one is `layer`.  The last fragments of a third are in registers and the next third is there: the one
    // after those in LDS is loaded in its place.
    auto turn = [&](auto st_c, int layer, int layer2) __attribute__((always_inline)) {
        constexpr int st = decltype(st_c)::value, k = st / 6;
        if constexpr (st % 6 == 4) {
            asm volatile("s_waitcnt vmcnt(%0)" :: "n"((SLOTS - 2) * (THIRD / 8192)) : "memory");
            barrier();
            if constexpr (SLOTS == 3) load_third(layer2, k, k);
            else if constexpr (k == 0) load_third(layer, 2, slot_of(0));
            else load_third(layer2, k - 1, slot_of(k));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto weights = [&](const uint8_t* (&wt)[3], int l) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 3; ++k) wt[k] = lds + slot_of(k) * THIRD + (mh << 11) + (l << 4);
    };
    auto bias_of = [&](f32x4 (&b)[2], int layer) __attribute__((always_inline)) {
        const int l = lane_now();
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const float4 v = *(const float4*)(a.bias + min(layer, a.layers - 1) * 64 + (mh * 2 + m) * 16 + (l >> 4) * 4);
            b[m][0] = v.x; b[m][1] = v.y; b[m][2] = v.z; b[m][3] = v.w;
        }
    };

#pragma unroll
    for (int k = 0; k < SLOTS; ++k) load_third(0, k, k);
    uint32_t done = 0;                                       // units of this workgroup so far
    for (int s = 0, u = wg; s < steps;) {
        const int n = u / cells_img, cy = (u - n * cells_img) / cells_x, y0 = cy * TH, cx = u - n * cells_img - cy * cells_x, x0 = cx * BODY_PAIR_COLS;
        int s_next = s, u_next = u + G;
        if (u_next >= units) { u_next = wg; ++s_next; }
        const bool two = 2 * s + 1 < a.layers;               // else the odd layer at the end
        const bool res = a.topology != RH_NET_PLAIN;         // two: + the unit's input; one: + the first conv's output
        const bool relu2 = !res;
        const __bf16* in = s ? out_of(s - 1) : a.h;
        // ---- all that needs no other unit ----
        f32x4 bias1[2], bias2[2];
        if (two) bias_of(bias1, 2 * s);
        bias_of(bias2, two ? 2 * s + 1 : 2 * s);
        // the patch begins two rows and two columns ahead of the unit.  Only the two rows and columns around the unit, where this workgroup made the rest
        const bool own = stay && s;
        uint32_t poff[NPW];
        int plds[NHW];
        const int l0 = lane_now(), t0 = wave * 64 + l0;
        if (own) {
#pragma unroll
            for (int i = 0; i < NHW; ++i) {
                const int p = i * 512 + t0, q = p >> 3, c = p & 7;                        // pixel q of: two rows above, two below, four columns
                const int e = q - 4 * PW, row = q < 2 * PW ? q / PW : e < 0 ? TH + q / PW : 2 + (e >> 2);
                const int px = e < 0 ? q % PW : (e & 3) + (e & 2 ? PW - 4 : 0), gy = y0 - 2 + row, gx = x0 - 2 + px;
                const bool ok = ((uint32_t)gy < (uint32_t)a.H) & ((uint32_t)gx < (uint32_t)a.W);
                poff[i] = ok ? (uint32_t)((gy * a.W + gx) * PIXB + (c << 4)) : OOB_OFF;
                plds[i] = (row * PW + px) * PIXB + ((c ^ (px & 7)) << 4);
            }
        } else
#pragma unroll
        for (int i = 0; i < NPW; ++i) {
            const int p = i * 512 + t0, row = p / (PW * 8), px = (p - row * (PW * 8)) >> 3, gy = y0 - 2 + row, gx = x0 - 2 + px;
            const bool ok = ((uint32_t)gy < (uint32_t)a.H) & ((uint32_t)gx < (uint32_t)a.W);
            poff[i] = ok ? (uint32_t)((gy * a.W + gx) * PIXB + (((p ^ px) & 7) << 4)) : OOB_OFF;
        }
        uint32_t kept1 = ~0u, kept2 = ~0u;                   // bit i: the lane's pixel of run i is inside the image (and kept)
        {
            const int wpr = (a.W + 31) >> 5, x1 = x0 - 1 + col_of(l0), x2 = x0 + col_of(l0);
            __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)(a.keep + (KEEP ? (size_t)n * a.H * wpr : 0)), 0, KEEP ? (uint32_t)(a.H * wpr) * 4u : 0u, RSRC_FLAGS);
            // words outside the image lie outside the descriptor's range, by their column or by their row, and read as zeros
            auto kept = [&](int y, int x, uint32_t at) __attribute__((always_inline)) {
                return __builtin_amdgcn_raw_buffer_load_b32(rk, at + ((uint32_t)y < (uint32_t)a.H ? (uint32_t)(y * wpr) * 4u : OOB_OFF), 0, 0) >> (x & 31) & 1u;
            };
            const uint32_t at1 = (uint32_t)x1 < (uint32_t)a.W ? (uint32_t)(x1 >> 5) * 4u : OOB_OFF >> 1, at2 = x2 < a.W ? (uint32_t)(x2 >> 5) * 4u : OOB_OFF >> 1;
            kept1 = 0; kept2 = 0;
#pragma unroll
            for (int i = 0; i < N1; ++i) {
                const int y = y0 - 1 + 2 * i + rp;
                kept1 |= (KEEP ? kept(y, x1, at1) : (uint32_t)(((uint32_t)y < (uint32_t)a.H) & ((uint32_t)x1 < (uint32_t)a.W))) << i;
            }
            if constexpr (KEEP)
#pragma unroll
                for (int i = 0; i < N2; ++i) kept2 |= kept(y0 + 2 * i + rp, x2, at2) << i;
        }
        // ---- every wave for itself: the 3 x 3 units around have done the step before ----
        if (s) {
            const int l = lane_now(), yy = cy + l / 3 - 1, xx = cx + l % 3 - 1;
            const bool look = l < 9 && yy >= 0 && yy < cells_y && xx >= 0 && xx < cells_x;
            const uint32_t* word = a.done + (size_t)(n * cells_img + (look ? yy * cells_x + xx : 0)) * BODY_PAIR_WORDS;
            int polls = 0;
            while (__builtin_amdgcn_ballot_w64(look && __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < (uint32_t)s) != 0) {
                if (__hip_atomic_load(s_lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) || ++polls > BODY_POLLS) {
                    __hip_atomic_store(s_lost, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    asm volatile("global_store_dword %0, %1, off sc0 sc1\n\ts_waitcnt vmcnt(0)" :: "v"(a.lost), "v"(1u) : "memory");
                    break;
                }
            }
        }
        {
            __amdgpu_buffer_rsrc_t rin = __builtin_amdgcn_make_buffer_rsrc((void*)(in + (size_t)n * img_elems), 0, img_bytes, RSRC_FLAGS);
            if (own) {
                i32x4 v[NHW];
#pragma unroll
                for (int i = 0; i < NHW; ++i) v[i] = __builtin_amdgcn_raw_buffer_load_b128(rin, poff[i], 0, LD_PAST);
#pragma unroll
                for (int i = 0; i < NHW; ++i) if (i < NHW - 1 || i * 512 + t0 < NH) *(i32x4*)(lds_p + plds[i]) = v[i];
            } else
#pragma unroll
            for (int i = 0; i < NPW; ++i) {
                if (i == NPW - 1 && i * 8 + wave >= NP) break;
                asm volatile("s_add_u32 m0, %0, %c1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen sc1 lds"
                             :: "s"(base), "n"(SLOTS * THIRD + i * 8192), "v"(poff[i]), "s"(rin) : "memory", "scc", "m0");
            }
        }
        // the skip of the odd layer
        uint4 skip[N2];
        const __amdgpu_buffer_rsrc_t rskip = __builtin_amdgcn_make_buffer_rsrc((void*)(a.h + (size_t)n * img_elems), 0, !two && res ? img_bytes : 0u, RSRC_FLAGS);
        const bool all = !stay || s + 1 == steps;            // else only what other units read
        auto out_off = [&](int i, int col, int grp) __attribute__((always_inline)) {
            const int y = y0 + 2 * i + rp, x = x0 + col;
            return (y < a.H) & (col < BODY_PAIR_COLS) & (x < a.W) ? (uint32_t)((y * a.W + x) * PIXB + (grp << 4)) : OOB_OFF;
        };
        if (!two)
#pragma unroll
            for (int i = 0; i < N2; ++i) {
                const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rskip, out_off(i, col_of(l0), grp_of(l0)), 0, LD_PAST);
                skip[i] = make_uint4(v[0], v[1], v[2], v[3]);
            }
        if (__hip_atomic_load(s_lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) bias2[0][0] = __builtin_nanf("");     // marks the result where no ReLU drops it
        lds_dma_wait();
        barrier();
        // ---- first layer ----
        if (two) {
            f32x4 acc[N1][2];
            auto hook = [&](auto st_c) __attribute__((always_inline)) { turn(st_c, 2 * s, 2 * s + 1); };
            const uint8_t* wt[3];
            const int l = lane_now();
            weights(wt, l);
            body_pair_products<N1>(acc, bias1, wt, rows, l, 0, hook);
            if (SLOTS == 2) par ^= 1;
            const int le = lane_now(), col = col_of(le), grp = grp_of(le), px = col + 2;
            const uint8_t* at = lds_p + ((rp + 2) * PW + px) * PIXB + ((grp ^ (px & 7)) << 4);
#pragma unroll
            for (int i = 0; i < N2; ++i) skip[i] = *(const uint4*)(at + i * (2 * PW * PIXB));
            barrier();                                       // nobody reads the patch any more
            uint8_t* to = lds_p + (rp * PW + col) * PIXB + ((grp ^ (col & 7)) << 4);
#pragma unroll
            for (int i = 0; i < N1; ++i) {
                uint2 p0 = conv64_round(acc[i][0]), p1 = conv64_round(acc[i][1]);
                p0.x = relu_bf16x2(p0.x); p0.y = relu_bf16x2(p0.y); p1.x = relu_bf16x2(p1.x); p1.y = relu_bf16x2(p1.y);
                uint4 v = body_pair_lanes(p0, p1);
                const uint32_t k = 0u - (kept1 >> i & 1u);
                v.x &= k; v.y &= k; v.z &= k; v.w &= k;
                *(uint4*)(to + i * (2 * PW * PIXB)) = v;
            }
            barrier();
        }
        // ---- second layer, or the odd one ----
        {
            f32x4 acc[N2][2];
            auto hook = [&](auto st_c) __attribute__((always_inline)) { turn(st_c, two ? 2 * s + 1 : 2 * s, 2 * s_next); };
            const uint8_t* wt[3];
            const int l = lane_now();
            weights(wt, l);
            body_pair_products<N2>(acc, bias2, wt, two ? rows : rows + PW * PIXB, l, two ? 0 : 1, hook);
            if (SLOTS == 2) par ^= 1;
            const int le = lane_now(), col = col_of(le), grp = grp_of(le);
            const bool side = all | (col < 2) | (col >= BODY_PAIR_COLS - 2);
            const __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc((void*)(out_of(s) + (size_t)n * img_elems), 0, img_bytes, RSRC_FLAGS);
#pragma unroll
            for (int i = 0; i < N2; ++i) {
                uint2 p0 = conv64_round(acc[i][0]), p1 = conv64_round(acc[i][1]);
                if (relu2) { p0.x = relu_bf16x2(p0.x); p0.y = relu_bf16x2(p0.y); p1.x = relu_bf16x2(p1.x); p1.y = relu_bf16x2(p1.y); }
                uint4 v = body_pair_lanes(p0, p1);
                if (res) {
                    v.x = pack_bf16x2(bf16_lo(v.x) + bf16_lo(skip[i].x), bf16_hi(v.x) + bf16_hi(skip[i].x));
                    v.y = pack_bf16x2(bf16_lo(v.y) + bf16_lo(skip[i].y), bf16_hi(v.y) + bf16_hi(skip[i].y));
                    v.z = pack_bf16x2(bf16_lo(v.z) + bf16_lo(skip[i].z), bf16_hi(v.z) + bf16_hi(skip[i].z));
                    v.w = pack_bf16x2(bf16_lo(v.w) + bf16_lo(skip[i].w), bf16_hi(v.w) + bf16_hi(skip[i].w));
                }
                if constexpr (KEEP) { const uint32_t k = 0u - (kept2 >> i & 1u); v.x &= k; v.y &= k; v.z &= k; v.w &= k; }
                const i32x4 o = {(int)v.x, (int)v.y, (int)v.z, (int)v.w};
                const uint32_t off = out_off(i, col, grp);
                __builtin_amdgcn_raw_buffer_store_b128(o, rout, (i == 0) | (i == N2 - 1) | side ? off : OOB_OFF, 0, ST_THROUGH);
                skip[i] = off == OOB_OFF ? make_uint4(0, 0, 0, 0) : v;
            }
        }
        barrier();                                           // nobody reads the tensor between any more
        const int lw = lane_now(), col = col_of(lw), grp = grp_of(lw);
        if (stay && s + 1 < steps && col < BODY_PAIR_COLS) {
            const int px = col + 2;
            uint8_t* at = lds_p + ((rp + 2) * PW + px) * PIXB + ((grp ^ (px & 7)) << 4);
#pragma unroll
            for (int i = 0; i < N2; ++i) *(uint4*)(at + i * (2 * PW * PIXB)) = skip[i];
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the stores are acknowledged, of all waves once the count is full
        if (lane == 0 && __hip_atomic_fetch_add(stored, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == done * 8 + 7)
            __hip_atomic_store(a.done + (size_t)u * BODY_PAIR_WORDS, (uint32_t)s + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ++done;
        s = s_next; u = u_next;
    }
    lds_dma_wait();
}
