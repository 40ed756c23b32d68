// 64 -> 64-channel-chunk bf16 conv3x3 on the matrix cores, two-team variant.
//
// Same implicit GEMM, patch layout and buffer addressing as k_conv_mfma (conv_mfma.hip), products and weight layout of
// conv_mfma64.h; the workgroup has 8 waves = two teams of 4.  The teams share the
// LDS-resident weights and own one 10 x 34 pixel patch each: a team computes one half (8 x 32
// pixels) of a 16 x 32 tile at a time.  The teams run one half apart: while one team is in its
// MFMA loop, the other rounds its finished accumulators to bf16, adds the skip tensor, writes
// the result, and puts its next patch into LDS.  Every SIMD holds one wave of each team, so the
// matrix pipe is fed by one wave while the other does vector-ALU, LDS and memory work.
//
// The hardware barrier counts all 8 waves, so both teams execute the same barrier sequence:
// time is cut into phases of exactly two barriers.
//   compute phase : sub-steps 0..MID-1 of conv64_products | barrier | sub-steps MID..17 | barrier
//                   (LDS fragment reads and MFMAs only: a wave that issues a wide global memory
//                   instruction cannot issue MFMAs for some 60-90 cycles, so the MFMA loop
//                   carries none)
//   drain phase   : issue the global loads (next patch, skip), accumulators -> bf16 -> own LDS
//                   slice -> registers, + skip, global stores | barrier |
//                   next patch registers -> LDS | barrier
// Team 0 runs compute, drain, compute, ...; team 1 starts with an idle phase, so the phases
// pair up.  The unit of work is the half tile (8 x 32 pixels): the halves are numbered 2 * tile +
// half and dealt out so that workgroup w takes units w, w + G, w + 2G, ... alternately with team 0
// and team 1 (G workgroups).  When the units do not divide evenly team 1 has one unit fewer than
// team 0 and ends with the idle phase instead (a whole tile per workgroup as the unit would leave
// half the chip idle for a full round whenever the tile count is not a multiple of G).  The
// number of phases depends only on kernel arguments, the workgroup index and - with a tile list -
// the list's length (never on anything that differs between the waves of a workgroup), the
// prefetch past a team's last unit loads out of range (zeros), and no wave leaves the loop
// early: every barrier is reached by all 8 waves.
#include <stdlib.h>

#include "conv_mfma64.h"

__device__ __forceinline__ void phase_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }
__device__ __forceinline__ void idle_phase() { phase_barrier(); phase_barrier(); }

// LIST: the half tiles to compute come from a.tile_list (box-masked mode) instead of being all of
// all images.  The entry of the next tile is requested with a vector load at the start of the
// compute phase and read at the start of the drain phase, a whole phase later: a scalar load would
// share its counter with the LDS fragment reads and turn their partial waits into full ones.
// KEEP (exact-border mode): an output pixel is written as zero where a.keep has no bit for it.  A wave's row of 32
// pixels is one word of the mask (half a word at twice its resolution), requested like the list entry.
template <bool SKIP, bool RELU, int MID, bool LIST, bool KEEP>
__global__ __launch_bounds__(512) void k_conv_mfma_duo(conv_args a)
{
    constexpr int CIN = 64, NCH = 8, PIXB = 128, TH = 8, PH = TH + 2, RW = 2;
    constexpr int WBYTES = 9 * CIN * CIN * 2, PATCHB = PH * PW * PIXB, NSTEP = C64_SUBSTEPS, CQ = 64;
    constexpr int NMAIN = PH, NHP = PH * 2 * NCH, NHALO = 1, NPRE = NMAIN + NHALO;      // 16-byte patch pieces per thread
    static_assert(NHP <= 256, "halo pieces must fit one per thread");
    static_assert(MID >= 1 && MID <= NSTEP - 1, "the compute phase must hold exactly two barriers");
    // MID: the compute phase's first barrier comes after MID of the 18 sub-steps; it pairs with the end
    // of the other team's loads + rounding + skip add + stores
    constexpr int NCHO = 8, OPIXB = 128, NOUT = RW * 32 * NCHO / 64, PPJ = 8, JPR = 4;   // output pieces per lane

    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    // team and wave are uniform over a wave: taken through readfirstlane so that the compiler keeps
    // everything derived from them (tile rows, row validity, descriptors) in scalar registers
    const int tid = threadIdx.x, ttid = tid & 255, lane = tid & 63;
    const int team = __builtin_amdgcn_readfirstlane(tid >> 8), wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
    uint8_t* lds_w = lds;
    uint8_t* lds_p = lds + WBYTES + team * PATCHB;
    float* lds_b = (float*)(lds + WBYTES + 2 * PATCHB);       // the chunk's 64 biases

    // requested first of all (behind the copy to LDS, which may write anything, it would be a vector load that waits for it)
    const uint32_t* counter = LIST ? a.n_list : a.n_valid;
    const uint32_t n_found = counter ? *counter : (uint32_t)a.N;
    // Tile order.  Workgroups go to the 8 XCDs round-robin; XCD x takes a contiguous run of tile
    // lanes so that neighbouring tiles (shared halo pixels) meet in one L2.
    // Layers with several output chunks (the upsampling convs): when the grid allows it the chunks
    // are dealt to workgroups instead of looped over - the n_chunks workgroups of one XCD that
    // share a tile lane process the same tiles at about the same time, each with its own chunk's
    // weights resident, so the input is fetched from HBM once and the other reads hit L2
    // (looping chunks outermost reads the whole input once per chunk).
    const bool deal = a.n_chunks > 1 && gridDim.x % (8 * a.n_chunks) == 0;
    const int G = deal ? gridDim.x / a.n_chunks : gridDim.x;                  // tile lanes
    const int xcd = blockIdx.x % 8, local = blockIdx.x / 8;
    const int chunk_begin = deal ? local % a.n_chunks : 0, chunk_end = deal ? chunk_begin + 1 : a.n_chunks;
    // The first chunk's weights depend on nothing that is read from memory: they are on their way to LDS before the
    // image count is known and the first patch can be asked for.  (Behind it, through registers, three pieces at a
    // time, they made four round trips in a row out of what are two.)
    auto load_weights = [&](int chunk) __attribute__((always_inline)) {
        lds_dma<512, WBYTES>(lds_w, a.wp + (size_t)chunk * (WBYTES / 16), team * 4 + wave, lane);
    };
    load_weights(chunk_begin);
    const int n_img = min((int)n_found, a.N);
    const int tiles_x = (a.W + 31) / 32, tiles_y = (a.H + 15) / 16;
    const int tiles_img = tiles_x * tiles_y;
    // half tiles; with a list, its entries are half tiles packed as RH_CELL_ENTRY(image, row of 8, column of 32)
    const int n_units = LIST ? (int)n_found : 2 * n_img * tiles_img;
    // Few units: one after the other to all XCDs.  In runs the XCDs work, in step, at addresses a power of two apart, on the
    // same memory channels (EDSR x4 on 128 x 128 bins, us, runs / this: 3 bins 395 / 343, 6: 647 / 475, 8: 529 / 509; 16: 767 / 803).
    const int wg = deal ? xcd * (G / 8) + local / a.n_chunks
                        : ((G % 8 == 0 && n_units > 2 * G) ? xcd * (G / 8) + local : (int)blockIdx.x);
    auto units_from = [&](int first) { return n_units > first ? (n_units - first + 2 * G - 1) / (2 * G) : 0; };
    const int u_first = wg + team * G;                         // this team's units: u_first, u_first + 2G, ...
    const int iters0 = units_from(wg), iters1 = units_from(wg + G);           // team 1 has as many as team 0 or one fewer
    const int iters = team ? iters1 : iters0;
    const int ps = a.ps;
    const uint32_t in_img_bytes = (uint32_t)a.H * a.W * PIXB;
    const uint32_t out_img_bytes = (uint32_t)(a.H * ps) * (a.W * ps) * OPIXB;

    // per-thread constants of the patch pieces (see k_conv_mfma)
    const int m_col = ttid >> 3, m_c = ttid & 7;
    const int m_goff = m_col * PIXB + m_c * 16;
    const uint32_t m_lds = (uint32_t)((1 + m_col) * PIXB + ((m_c ^ ((1 + m_col) & 7)) << 4));
    const int h_row = ttid >> 4, h_side = (ttid >> 3) & 1, h_c = ttid & 7;     // halo piece (ttid < NHP)
    const int lcol = lane >> 3, lc = lane & 7;
    const int o_lane = (lcol * ps) * OPIXB + lc * 16;
    const int o_rowpitch = a.W * ps * OPIXB;
    const int row_pitch = a.W * PIXB;

    // origin of half `half` of tile number `tile` (rows y0..y0+7), image index n
    auto decode = [&](int tile, int half, int& n, int& y0, int& x0) __attribute__((always_inline)) {
        n = tile / tiles_img;
        const int tr = tile - n * tiles_img, ty = tr / tiles_x, tx = tr - ty * tiles_x;
        y0 = ty * 16 + half * TH; x0 = tx * 32;
    };
    // Consecutive layers walk the tensor in opposite directions: what a layer touched last (the
    // end of its input and output) is what the next layer touches first, while it is still in
    // the memory-side cache.  Walking every layer front to back through buffers that together
    // exceed that cache evicts each line just before it is needed again.
    __amdgpu_buffer_rsrc_t rlist = __builtin_amdgcn_make_buffer_rsrc((void*)a.tile_list, 0, LIST ? (uint32_t)n_units * 4u : 0u, RSRC_FLAGS);
    auto walk = [&](int u) __attribute__((always_inline)) { return (a.rev && u < n_units) ? n_units - 1 - u : u; };
    auto list_load = [&](int u) __attribute__((always_inline)) {         // list entry of unit u (0 past the end)
        return __builtin_amdgcn_raw_buffer_load_b32(rlist, u < n_units ? (uint32_t)walk(u) * 4u : OOB_OFF, 0, 0);
    };
    auto decode_cell = [&](int cell, int& n, int& y0, int& x0) __attribute__((always_inline)) {
        n = (int)((uint32_t)cell >> 16); y0 = (int)(((uint32_t)cell >> 7) & 511u) * TH; x0 = (int)((uint32_t)cell & 127u) * 32;
    };
    auto unit_origin = [&](int u, int& n, int& y0, int& x0) __attribute__((always_inline)) {
        if constexpr (LIST) decode_cell(__builtin_amdgcn_readfirstlane(list_load(u)), n, y0, x0);
        else { const int uu = walk(u); decode(uu >> 1, uu & 1, n, y0, x0); }
    };
    uint4 pre[NPRE];
    auto load_piece = [&](int j, __amdgpu_buffer_rsrc_t rin, int y0, int x0) __attribute__((always_inline)) {
        int off; bool ok;
        if (j < NMAIN) {
            const int gy = y0 - 1 + j;
            ok = gy >= 0 && gy < a.H && x0 + m_col < a.W;
            off = ((y0 - 1) * a.W + x0) * PIXB + m_goff + j * row_pitch;
        } else {
            const int gy = y0 - 1 + h_row, hx = h_side ? x0 + 32 : x0 - 1;
            ok = ttid < NHP && gy >= 0 && gy < a.H && hx >= 0 && hx < a.W;
            off = (gy * a.W + hx) * PIXB + h_c * 16;
        }
        const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rin, ok ? (uint32_t)off : OOB_OFF, 0, 0);
        pre[j] = make_uint4(v[0], v[1], v[2], v[3]);
    };
    auto store_patch = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NMAIN; ++j) *(uint4*)(lds_p + j * (PW * PIXB) + m_lds) = pre[j];
        const int px = h_side ? PW - 1 : 0;
        if (ttid < NHP) *(uint4*)(lds_p + (h_row * PW + px) * PIXB + ((h_c ^ (px & 7)) << 4)) = pre[NMAIN];
    };
    auto out_off = [&](int j, int y0, int x0, int si, int sj) __attribute__((always_inline)) {
        const int y = y0 + wave * RW + j / JPR, xb = x0 + (j % JPR) * PPJ;
        const bool ok = y < a.H && xb + lcol < a.W;
        const int off = (y * ps + si) * o_rowpitch + (xb * ps + sj) * OPIXB + o_lane;
        return ok ? (uint32_t)off : OOB_OFF;
    };
    auto in_rsrc = [&](int u, int n) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)(a.in + (size_t)n * a.H * a.W * CIN), 0,
                                                 u < n_units ? in_img_bytes : 0u, RSRC_FLAGS);
    };

    int cn = 0, cy0 = 0, cx0 = 0;                          // LIST: origin of the tile about to be computed
    float bias = 0.0f;
    auto first_patch = [&](int chunk) __attribute__((always_inline)) {         // requests it, of both teams
        if (tid < CQ) bias = a.bias[chunk * CQ + tid];
        unit_origin(u_first, cn, cy0, cx0);
        __amdgpu_buffer_rsrc_t rin = in_rsrc(u_first, u_first < n_units ? cn : 0);
#pragma unroll
        for (int j = 0; j < NPRE; ++j) load_piece(j, rin, cy0, cx0);
    };
    first_patch(chunk_begin);                              // ahead of the loops: ahead of what the compiler computes for all of their turns
    for (int chunk = chunk_begin; chunk < chunk_end; ++chunk) {
        if (chunk != chunk_begin) {
            __syncthreads();                               // all 8 waves: previous chunk completely done
            load_weights(chunk);
            first_patch(chunk);
        }
        if (tid < CQ) lds_b[tid] = bias;
        store_patch();
        lds_dma_wait();
        const int si = chunk / ps, sj = chunk - si * ps;
        __syncthreads();

        // Accumulators start from the bias: lane holds channels m*32 + 8*q + 4*hi + {0..3} in [m][4q..4q+3].  It stays in
        // 32 registers and is the first product's C operand; written into the accumulators anew for every unit (8 LDS
        // reads, 64 moves) it took both phases' time: 16 whole frames 5193 us a step, now 5147, the headline batch 2781, now 2760.
        conv64_acc acc;
        f32x4 bias_c[4];
        conv64_bias(bias_c, lds_b, lane);
        if (team == 1) idle_phase();
        for (int it = 0; it < iters; ++it) {
            const int unit = u_first + it * 2 * G, nunit = unit + 2 * G;
            int n, y0, x0, next_entry = 0;
            if constexpr (LIST) { n = cn; y0 = cy0; x0 = cx0; next_entry = list_load(nunit); }
            else unit_origin(unit, n, y0, x0);
            __amdgpu_buffer_rsrc_t rsk = __builtin_amdgcn_make_buffer_rsrc(
                (void*)((uint8_t*)a.skip + (size_t)n * out_img_bytes), 0, SKIP ? out_img_bytes : 0u, RSRC_FLAGS);
            uint4 sk[SKIP ? NOUT : 1];
            uint32_t kw[RW];
            if constexpr (KEEP) {
                const int rows = a.H >> a.keep_sh, wpr = ((a.W >> a.keep_sh) + 31) >> 5;
                __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)(a.keep + (size_t)n * rows * wpr), 0, (uint32_t)(rows * wpr) * 4u, RSRC_FLAGS);
#pragma unroll
                for (int r = 0; r < RW; ++r)
                    kw[r] = __builtin_amdgcn_raw_buffer_load_b32(rk, (uint32_t)((((y0 + wave * RW + r) >> a.keep_sh) * wpr + (x0 >> (5 + a.keep_sh))) * 4), 0, 0);
            }
            // ---------------- compute phase ----------------
            auto hook = [&](auto st_c) __attribute__((always_inline)) {
                constexpr int st = decltype(st_c)::value;
                if constexpr (SKIP && st % 3 != 0 && st * 2 / 3 < NOUT) {
                    constexpr int j = st * 2 / 3;
                    const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsk, out_off(j, y0, x0, 0, 0), 0, 0);
                    sk[j] = make_uint4(v[0], v[1], v[2], v[3]);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (LIST && st == MID - 1) {              // the next unit's list entry has long arrived: decode it here,
                    decode_cell(__builtin_amdgcn_readfirstlane(next_entry), cn, cy0, cx0);   // off the drain phase's critical path
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (st == MID - 1 || st == NSTEP - 1) {   // the two barriers of the compute phase
                    asm volatile("s_barrier" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            __builtin_amdgcn_s_setprio(2);             // the wave feeding the matrix pipe goes first
            conv64_products(acc, bias_c, lds_w + (lane << 4), lds_p + wave * RW * (PW * PIXB), lane, hook);
            __builtin_amdgcn_s_setprio(0);

            // ---------------- drain phase ----------------
            int nn, ny0, nx0;
            if constexpr (LIST) { nn = cn; ny0 = cy0; nx0 = cx0; }
            else unit_origin(nunit, nn, ny0, nx0);
            __amdgpu_buffer_rsrc_t rin = in_rsrc(nunit, nunit < n_units ? nn : 0);
            __amdgpu_buffer_rsrc_t rout = __builtin_amdgcn_make_buffer_rsrc(
                (void*)((uint8_t*)a.out + (size_t)n * out_img_bytes), 0, out_img_bytes, RSRC_FLAGS);
            // The global loads of the next tile's patch (stored to LDS at the end of the phase) are
            // issued here, by waves that are not feeding the matrix pipe.  The skip variant's
            // drain phase is the longer of the two phases: there the tile's skip values are loaded
            // during its own compute phase instead (one load after each of the first 8 steps), which
            // costs the matrix pipe a few issue slots but takes their issue time and their whole
            // latency off the critical phase.  The CU's one address unit
            // takes about 16 cycles per 64 x 16-byte instruction and all four waves of the team
            // arrive together, so a wave that issues its loads back to back is held for 60-90
            // cycles by each of them: the loads are dealt out one or two at a time between the
            // 16 units of rounding work instead.
            constexpr int NUNIT = 16;
            uint8_t* stg = lds_p + wave * (RW * 32 * OPIXB);
#pragma unroll
            for (int u = 0; u < NUNIT; ++u) {
                const int m = u >> 2, n = u >> 1 & 1, r = u & 1;
#pragma unroll
                for (int i = u * NPRE / NUNIT; i < (u + 1) * NPRE / NUNIT; ++i) load_piece(i, rin, ny0, nx0);
                uint2 pk = conv64_round(acc.v[r][n][m]);
                if constexpr (RELU) { pk.x = relu_bf16x2(pk.x); pk.y = relu_bf16x2(pk.y); }   // rounding keeps the sign
                *(uint2*)(stg + conv64_slot(r, n, m, lane)) = pk;
                __builtin_amdgcn_sched_barrier(0);
            }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the slice is private to the wave: no barrier
            uint4 ov[NOUT];
#pragma unroll
            for (int j = 0; j < NOUT; ++j) {
                const int r = j / JPR, px = (j % JPR) * PPJ + lcol;
                ov[j] = *(const uint4*)(stg + (r * 32 + px) * OPIXB + ((lc ^ (px & 7)) << 4));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NOUT; ++j) {
                uint4 o = ov[j];
                if constexpr (SKIP) {
                    o.x = pack_bf16x2(bf16_lo(o.x) + bf16_lo(sk[j].x), bf16_hi(o.x) + bf16_hi(sk[j].x));
                    o.y = pack_bf16x2(bf16_lo(o.y) + bf16_lo(sk[j].y), bf16_hi(o.y) + bf16_hi(sk[j].y));
                    o.z = pack_bf16x2(bf16_lo(o.z) + bf16_lo(sk[j].z), bf16_hi(o.z) + bf16_hi(sk[j].z));
                    o.w = pack_bf16x2(bf16_lo(o.w) + bf16_lo(sk[j].w), bf16_hi(o.w) + bf16_hi(sk[j].w));
                }
                if constexpr (KEEP) {
                    const uint32_t at = ((uint32_t)x0 >> a.keep_sh & 31u) + ((uint32_t)((j % JPR) * PPJ + lcol) >> a.keep_sh);
                    const uint32_t m = 0u - (kw[j / JPR] >> at & 1u);
                    o.x &= m; o.y &= m; o.z &= m; o.w &= m;
                }
                const i32x4 v = {(int)o.x, (int)o.y, (int)o.z, (int)o.w};
                __builtin_amdgcn_raw_buffer_store_b128(v, rout, out_off(j, y0, x0, si, sj), 0, ST_THROUGH);
                if constexpr (SKIP) __builtin_amdgcn_sched_barrier(0);
            }
            phase_barrier();                                  // 1: every wave of the team has read its slice back
            store_patch();                                    // next tile's patch (zeros after the last tile)
            phase_barrier();                                  // 2
        }
        // team 0's last drain phase pairs with team 1's last one, or - team 1 a unit short - with its idle phase
        if (team == 0 ? iters1 == iters0 : iters1 < iters0) idle_phase();
    }
}

template <bool SKIP, bool RELU, int MID, bool LIST, bool KEEP = false>
static hipError_t launch_duo(hipStream_t stream, int device, const conv_args& a, int grid)
{
    constexpr int lds = 9 * 64 * 64 * 2 + 2 * 10 * PW * 128 + 256;
    static bool attr_done[RH_MAX_DEVICES] = {};            // the attribute is per device
    if (!attr_done[device]) {
        hipError_t e = hipFuncSetAttribute((const void*)k_conv_mfma_duo<SKIP, RELU, MID, LIST, KEEP>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_done[device] = true;
    }
    hipLaunchKernelGGL((k_conv_mfma_duo<SKIP, RELU, MID, LIST, KEEP>), dim3(grid), dim3(512), lds, stream, a);
    return hipGetLastError();
}

hipError_t rh_launch_conv_duo(hipStream_t stream, int device, const conv_args& a, int grid, bool skip, bool relu)
{
    // first barrier of the compute phase after 15 of the 18 sub-steps (headline batch, us, 14 / 15 / 16: 2788 / 2784 / 2797)
    constexpr int MID = 15;
    if (a.tile_list) {
        if (a.n_chunks != 1) return hipErrorInvalidValue;      // a tile list goes with single-chunk layers only
        if (skip) return launch_duo<true, false, MID, true>(stream, device, a, grid);
        if (relu) return launch_duo<false, true, MID, true>(stream, device, a, grid);
        return launch_duo<false, false, MID, true>(stream, device, a, grid);
    }
    if (a.keep) {
        if (skip) return launch_duo<true, false, MID, false, true>(stream, device, a, grid);
        if (relu) return launch_duo<false, true, MID, false, true>(stream, device, a, grid);
        return launch_duo<false, false, MID, false, true>(stream, device, a, grid);
    }
    if (skip) return launch_duo<true, false, MID, false>(stream, device, a, grid);
    if (relu) return launch_duo<false, true, MID, false>(stream, device, a, grid);
    return launch_duo<false, false, MID, false>(stream, device, a, grid);
}
