// The body of a 64-channel bf16 net - every 3x3 conv between the first one and the tail - in ONE launch.
//
// A few images go two layers at a time (conv_body_pairs.h), more of them a layer at a time, as follows.
//
// A unit of work is one half tile (8 x 32 pixels, all 64 output channels) of one layer; it is computed as in
// k_conv_mfma_duo: two teams of four waves, one in its MFMA loop while the other rounds, stores and loads, in phases of
// two barriers.  What differs is where units come from and what they wait for:
//   - Units are numbered layer by layer; workgroup w of G takes units w, w + G, w + 2G, ..., with its two teams in turn, so
//     that the team about to compute always holds the earlier one.
//   - A unit of layer l reads the 3 x 3 half tiles around its own of layer l - 1.  Every wave that has stored its rows of
//     a unit writes l + 1 into a word of its own (`done`, four a half tile), and a unit starts when the 36 words around it
//     say so.  Buffers that are written again (t by every block, a in place) need no more than that: whoever read the old
//     values lies among the same 3 x 3 half tiles of the layer before.
//   - Workgroups sit on eight XCDs with an L2 each: activations and words are stored through (sc1) and loaded past (sc1)
//     the L2, and a wave's stores are acknowledged (vmcnt 0) before its word is written.
//   - Only workgroups that run take part: each signs the roll when it starts, and the roll closes when all have, or
//     BODY_ROLL_POLLS later, where other kernels hold compute units; who comes after that leaves at once (conv_body_roll.h).
//   - A wait for words is given up after BODY_POLLS looks, and every later one of the workgroup after one, so that the launch ends
//     whatever happens; the host is told by a word in its memory, and the next call fails (rh_check_lost).
// So every wait ends, whatever else the GPU runs: a unit waits for units with smaller numbers only, all in the hands of
// workgroups that run, and the smallest one not done does not wait.  Its team stores it and writes its words ahead of the
// phase's first barrier where the team beside it may be waiting inside that phase, and is the next to compute otherwise.
//
// Is a unit ready?  Wave 0 looks in the middle of the team's compute phase before it, so that the patch can be requested at
// the start of the drain phase; looks again during that phase, and requests the patch at its end; and at last all four
// waves look at the start of the unit's own compute phase until it is.  The first is what happens with six units or more a
// layer and workgroup, the last with one or two.
//
// What bounds it: with two or three units a workgroup and layer still the chain per layer of look, patch, 2 us of MFMAs, rounding, stores and words; with many the matrix pipe at the chip's power
// limit, as in k_conv_mfma_duo.  A layer's weights (72 KB) go to LDS while the other team stores.
#define LD_PAST 16                       // loads: sc1
#define BODY_ROLL_POLLS 64               // of about a us each
#define BODY_POLLS (1 << 21)             // a second or more: never reached while the workgroups on the roll run
#include "conv_body_pairs.h"
#include "conv_body_roll.h"

#define FEW_UNITS 4

__device__ __forceinline__ void body_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

struct body_unit { int layer, idx, n, y0, x0; };            // idx: its number in the layer

template <bool KEEP>
__global__ __launch_bounds__(512) void k_conv_mfma_body(body_args args)
{
    extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
    __shared__ uint32_t s_ready[2][2];                        // [team][its units in turn]: what it reads was there
    __shared__ uint32_t s_again[2], s_sync[2], s_lost, s_wg[3], s_stored;
    const int tid = threadIdx.x;
    int n_img = max(args.n_valid ? min((int)*args.n_valid, args.N) : args.N, 0);
    if (n_img == 0) return;                                  // nothing to do, or another way's to do
    const int pair_rows = body_pair_rows(n_img, args.H, args.W, gridDim.x);

    // ---- start: who takes part ----
    if (tid == 0) {
        const uint32_t units = pair_rows ? (uint32_t)body_pair_units(n_img, args.H, args.W, pair_rows) : (uint32_t)(n_img * ((args.W + 31) / 32) * ((args.H + 7) / 8));
        s_lost = 0; s_stored = 0; s_again[0] = 0; s_again[1] = 0; s_sync[0] = 0; s_sync[1] = 0; s_ready[0][0] = 0; s_ready[1][0] = 0;
        const uint32_t sign = __hip_atomic_fetch_add(args.roll, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        body_place p;
        for (int polls = 0;;) {
            uint32_t r = __hip_atomic_load(args.roll, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (body_roll_place(sign, r, gridDim.x, blockIdx.x, &p)) break;
            if (++polls > BODY_ROLL_POLLS)
                __hip_atomic_compare_exchange_strong(args.roll, &r, body_roll_closed(r), __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        body_roll_spread(&p, gridDim.x, units);
        s_wg[2] = body_roll_leaves(&p, units);
        s_wg[0] = p.wg; s_wg[1] = p.G;
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(s_wg[2])) return;     // not needed, or too late
    int G = (int)__builtin_amdgcn_readfirstlane(s_wg[1]), wg = (int)__builtin_amdgcn_readfirstlane(s_wg[0]);
    switch (pair_rows) {
#define PAIRS(TH) case TH: body_pairs<TH, KEEP>(lds, &s_stored, &s_lost, n_img, wg, G); return
    PAIRS(4); PAIRS(6); PAIRS(8); PAIRS(10); PAIRS(12); PAIRS(14); PAIRS(16); PAIRS(18); PAIRS(20); PAIRS(22);
#undef PAIRS
    }
    const body_args a = body_args_anew(n_img, wg, G);
    constexpr int CIN = 64, NCH = 8, PIXB = 128, TH = 8, PH = TH + 2, RW = 2;
    constexpr int WBYTES = 9 * CIN * CIN * 2, PATCHB = PH * PW * PIXB, NSTEP = C64_SUBSTEPS, MID = 15;
    constexpr int NMAIN = PH, NHP = PH * 2 * NCH, NPRE = NMAIN + 1;
    constexpr int NOUT = 8, PPJ = 8, JPR = 4;
    static_assert(NHP <= 256, "halo pieces must fit one per thread");

    const int ttid = tid & 255, lane = tid & 63;
    const int team = __builtin_amdgcn_readfirstlane(tid >> 8), wave = __builtin_amdgcn_readfirstlane((tid >> 6) & 3);
    uint8_t* lds_w = lds;
    uint8_t* lds_p = lds + WBYTES + team * PATCHB;
    __shared__ __attribute__((aligned(16))) float s_bias[2][64];

    const int cells_x = (a.W + 31) / 32, cells_y = (a.H + TH - 1) / TH, cells_img = cells_x * cells_y;
    const int layer_units = n_img * cells_img;
    const uint32_t img_bytes = (uint32_t)a.H * a.W * PIXB;
    const int row_pitch = a.W * PIXB;
    const size_t img_elems = (size_t)a.H * a.W * CIN;

    // what layer l reads and writes (the order of the buffers is the caller's of one launch per layer)
    const bool plain = a.topology == RH_NET_PLAIN;
    auto layer_skips = [&](int l) __attribute__((always_inline)) { return !plain && ((l & 1) || (a.topology == RH_NET_EDSR && l == a.layers - 1)); };
    auto layer_relu = [&](int l) __attribute__((always_inline)) { return !layer_skips(l); };
    auto layer_in = [&](int l) __attribute__((always_inline)) { return plain ? (l == 0 ? a.h : (l & 1) ? a.a : a.t) : (l & 1) ? a.t : l == 0 ? a.h : a.a; };
    auto layer_out = [&](int l) __attribute__((always_inline)) { return plain ? ((l & 1) ? a.t : a.a) : (l & 1) ? a.a : a.t; };
    auto layer_skip = [&](int l) __attribute__((always_inline)) { return (l & 1) && l != 1 ? a.a : a.h; };       // l = 1 and the body's end: h

    // Where a lane reads and writes is worked out anew in every phase (`lane` and `ttid` pass through an empty asm
    // statement there): kept over the loop these addresses would not fit the registers.  With some of them kept, 11 registers (exact-border
    // mode: 24) lay in scratch memory, from where every unit loaded them again, and 275 (506) scalars in lanes of others: EDSR x2 of 8 blocks
    // on 128 x 128 bins, us, so / now, 9 bins 242 / 228, 12: 277 / 267, 16: 354 / 338, 20: 397 / 394.
    uint4 pre[NPRE];
    auto load_piece = [&](int j, int tt, __amdgpu_buffer_rsrc_t rin, int y0, int x0) __attribute__((always_inline)) {
        const int m_col = tt >> 3, m_goff = m_col * PIXB + (tt & 7) * 16;
        const int h_row = tt >> 4, h_side = (tt >> 3) & 1, h_c = tt & 7;       // halo piece (tt < NHP)
        int off; bool ok;
        if (j < NMAIN) {
            const int gy = y0 - 1 + j;
            ok = ((uint32_t)gy < (uint32_t)a.H) & (x0 + m_col < a.W);
            off = ((y0 - 1) * a.W + x0) * PIXB + m_goff + j * row_pitch;
        } else {
            const int gy = y0 - 1 + h_row, hx = h_side ? x0 + 32 : x0 - 1;
            ok = (tt < NHP) & ((uint32_t)gy < (uint32_t)a.H) & ((uint32_t)hx < (uint32_t)a.W);
            off = (gy * a.W + hx) * PIXB + h_c * 16;
        }
        const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rin, ok ? (uint32_t)off : OOB_OFF, 0, LD_PAST);
        pre[j] = make_uint4(v[0], v[1], v[2], v[3]);
    };
    auto store_patch = [&](int tt) __attribute__((always_inline)) {
        const int m_col = tt >> 3, m_c = tt & 7, h_row = tt >> 4, h_side = (tt >> 3) & 1, h_c = tt & 7;
        const uint32_t m_lds = (uint32_t)((1 + m_col) * PIXB + ((m_c ^ ((1 + m_col) & 7)) << 4));
#pragma unroll
        for (int j = 0; j < NMAIN; ++j) *(uint4*)(lds_p + j * (PW * PIXB) + m_lds) = pre[j];
        const int px = h_side ? PW - 1 : 0;
        if (tt < NHP) *(uint4*)(lds_p + (h_row * PW + px) * PIXB + ((h_c ^ (px & 7)) << 4)) = pre[NMAIN];
    };
    auto out_off = [&](int j, int ln, int y0, int x0) __attribute__((always_inline)) {
        const int lcol = ln >> 3, o_lane = lcol * PIXB + (ln & 7) * 16;
        const int y = y0 + wave * RW + j / JPR, xb = x0 + (j % JPR) * PPJ;
        const bool ok = (y < a.H) & (xb + lcol < a.W);
        return ok ? (uint32_t)(y * row_pitch + xb * PIXB + o_lane) : OOB_OFF;
    };
    auto rsrc_of = [&](const __bf16* base, int n, bool on) __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)(base + (size_t)n * img_elems), 0, on ? img_bytes : 0u, RSRC_FLAGS);
    };
    auto lane_now = [&]() __attribute__((always_inline)) { int l = lane; asm volatile("" : "+v"(l)); return l; };
    // unit number `u` places behind; layer = a.layers: there is none
    auto unit_at = [&](int layer, int idx, int ahead) __attribute__((always_inline)) {
        body_unit u;
        idx += ahead;
        while (idx >= layer_units && layer < a.layers) { idx -= layer_units; ++layer; }
        u.layer = layer; u.idx = idx;
        u.n = a.img_magic ? (int)__umulhi((uint32_t)idx, a.img_magic) : idx;
        const int c = idx - u.n * cells_img, cy = a.row_magic ? (int)__umulhi((uint32_t)c, a.row_magic) : c;
        u.y0 = cy * TH; u.x0 = (c - cy * cells_x) * 32;
        return u;
    };
    // the words around a unit: lane j < 36 has word j % 4 of half tile j / 4 of the 3 x 3 around it
    auto load_words = [&](const body_unit& u) __attribute__((always_inline)) {
        const int l = lane_now(), j = l >> 2, cy = u.y0 / TH + j / 3 - 1, cx = u.x0 / 32 + j % 3 - 1;
        const bool in = l < 36 && cy >= 0 && cy < cells_y && cx >= 0 && cx < cells_x && u.layer > 0 && u.layer < a.layers;
        return in ? __hip_atomic_load(a.done + ((size_t)u.n * cells_img + cy * cells_x + cx) * 4 + (l & 3), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                  : 0x7FFFFFFFu;
    };
    // all four waves of a team have come here (their LDS writes are done)
    uint32_t sync_no = 0;
    auto team_sync = [&]() __attribute__((always_inline)) {
        sync_no += 4;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (lane == 0) __hip_atomic_fetch_add(&s_sync[team], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        while ((int)(__builtin_amdgcn_readfirstlane(__hip_atomic_load(&s_sync[team], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) - sync_no) < 0)
            __builtin_amdgcn_s_sleep(1);
        asm volatile("" ::: "memory");
    };
    int bias_layer = -1;                                     // layer whose biases lie in s_bias[team]
    auto load_bias = [&](int l) __attribute__((always_inline)) { return wave == 0 ? a.bias[l * 64 + lane_now()] : 0.0f; };
    auto store_bias = [&](float v) __attribute__((always_inline)) { if (wave == 0) s_bias[team][lane_now()] = v; };

    // A wave of the workgroup has given up a wait.
    auto lost = [&]() __attribute__((always_inline)) { return __hip_atomic_load(&s_lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    // As a store that the compiler sees in the loop of units it would have it wait for all loads there (40 bins 1585 -> 1620 us).
    auto tell_host = [&]() __attribute__((always_inline)) {
        asm volatile("global_store_dword %0, %1, off sc0 sc1\n\ts_waitcnt vmcnt(0)" :: "v"(a.lost), "v"(1u) : "memory");
    };

    body_unit cur = unit_at(0, wg, team * G);                // the unit to compute next
    body_unit prev = cur;                                    // the one in the accumulators
    bool loaded = false, word_due = false;
    int resident = -1;                                       // layer whose weights are in LDS

    auto mark_done = [&](const body_unit& u) __attribute__((always_inline)) {
        if (lane == 0)
            __hip_atomic_store(a.done + ((size_t)u.n * cells_img + (u.y0 / TH) * cells_x + u.x0 / 32) * 4 + wave, (uint32_t)u.layer + 1u,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };

    // A unit's two phases: computes `cur`, then - while the other team computes - stores it, and fetches the next one's
    // patch where that is ready.  True: the last.
    int turn = 0;                                            // units of this team so far
    // FEW: no look from the compute phase and no early patch.  With up to FEW_UNITS units a workgroup and layer neither is in time,
    // and the 11 loads of no bytes stood in the way of the words that others wait for: EDSR x4 on 128 x 128 bins, us, with them / without,
    // 9 bins 492 / 444, 10: 486 / 459, 12: 521 / 512, 16: 658 / 643, 18, 4.5 units: 710 / 732, 24: 912 / 948; 30 of 96 x 96, 4.2: 675 / 685.
    auto unit = [&](auto skip_c, auto few_c) __attribute__((always_inline)) -> bool {
        constexpr bool SKIP = decltype(skip_c)::value, FEW = decltype(few_c)::value;
        conv64_acc acc;
        uint4 sk[SKIP ? NOUT : 1];
        uint32_t kw[KEEP ? RW : 1];
        body_unit nu;
        int front_layer = 0;
        {
        const int y0 = cur.y0, x0 = cur.x0;
        int ln = lane;
        asm volatile("" : "+v"(ln));
        __amdgpu_buffer_rsrc_t rsk = rsrc_of(layer_skip(cur.layer), cur.n, SKIP);
        if constexpr (KEEP) {
            const int wpr = (a.W + 31) >> 5;
            __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)(a.keep + (size_t)cur.n * a.H * wpr), 0, (uint32_t)(a.H * wpr) * 4u, RSRC_FLAGS);
#pragma unroll
            for (int r = 0; r < RW; ++r) kw[r] = __builtin_amdgcn_raw_buffer_load_b32(rk, (uint32_t)(((y0 + wave * RW + r) * wpr + (x0 >> 5)) * 4), 0, 0);
        }
        f32x4 bias_c[4];
        conv64_bias(bias_c, s_bias[team], ln);
        uint32_t words = 0;
        auto hook = [&](auto st_c) __attribute__((always_inline)) {
            constexpr int st = decltype(st_c)::value;
            if constexpr (SKIP && st % 3 != 0 && st * 2 / 3 < NOUT) {
                constexpr int j = st * 2 / 3;
                const i32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsk, out_off(j, ln, y0, x0), 0, LD_PAST);
                sk[j] = make_uint4(v[0], v[1], v[2], v[3]);
                __builtin_amdgcn_sched_barrier(0);
            }
            // is what the team's next unit reads there?  Both teams know after the phase's end
            if constexpr (st == 3) {
                nu = unit_at(cur.layer, cur.idx, 2 * G);
                front_layer = cur.layer + (cur.idx + G >= layer_units ? 1 : 0);        // G <= layer_units
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (st == 8) {
                if (word_due) {                              // the last unit's stores were made a phase ago: all but the loads since then are done
                    asm volatile("s_waitcnt vmcnt(%0)" :: "n"((SKIP ? 6 : 0) + (KEEP ? RW : 0)) : "memory");
                    mark_done(prev);
                }
                if (!FEW && wave == 0) words = load_words(nu);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (st == NSTEP - 2) {
                if (!FEW && wave == 0) {
                    const bool ready = __builtin_amdgcn_ballot_w64(words >= (uint32_t)nu.layer) == ~0ull;
                    if (lane == 0) s_ready[team][(turn & 1) ^ 1] = ready;
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (st == NSTEP - 1) { if (wave == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
            if constexpr (st == MID - 1 || st == NSTEP - 1) {
                asm volatile("s_barrier" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        __builtin_amdgcn_s_setprio(2);
        conv64_products(acc, bias_c, lds_w + (ln << 4), lds_p + wave * RW * (PW * PIXB), ln, hook);
        __builtin_amdgcn_s_setprio(0);
        }
        // ---------------- the other team computes ----------------
        const uint32_t ready0 = FEW ? 0u : s_ready[team ^ 1][(turn + team) & 1], ready1 = FEW ? 0u : s_ready[team][(turn & 1) ^ 1];
        uint32_t again = 0;
        const bool at_end = front_layer >= a.layers;
        const bool none = nu.layer >= a.layers, early = !none && __builtin_amdgcn_readfirstlane(ready1);
        bool fetch = early;
        if (!early && wave == 0) again = load_words(nu);
        {
        const int y0 = cur.y0, x0 = cur.x0;
        int ln = lane;
        asm volatile("" : "+v"(ln));
        const int lcol = ln >> 3, lc = ln & 7, tt = wave * 64 + ln;
        __amdgpu_buffer_rsrc_t rin = rsrc_of(layer_in(nu.layer), early ? nu.n : 0, early);      // a range of 0 reads nothing: no branches, which would have the compiler wait for all loads
        __amdgpu_buffer_rsrc_t rout = rsrc_of(layer_out(cur.layer), cur.n, true);
        constexpr int NUNIT = 16;
        uint8_t* stg = lds_p + wave * (RW * 32 * PIXB);
#pragma unroll
        for (int u = 0; u < NUNIT; ++u) {
            const int m = u >> 2, n = u >> 1 & 1, r = u & 1;
#pragma unroll
            for (int i = u * NPRE / NUNIT; i < (u + 1) * NPRE / NUNIT && !FEW; ++i) load_piece(i, tt, rin, nu.y0, nu.x0);
            uint2 pk = conv64_round(acc.v[r][n][m]);
            if constexpr (!SKIP) { pk.x = relu_bf16x2(pk.x); pk.y = relu_bf16x2(pk.y); }
            *(uint2*)(stg + conv64_slot(r, n, m, ln)) = pk;
            __builtin_amdgcn_sched_barrier(0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // the slice is private to the wave: no barrier
        uint4 ov[NOUT];
#pragma unroll
        for (int j = 0; j < NOUT; ++j) {
            const int r = j / JPR, px = (j % JPR) * PPJ + lcol;
            ov[j] = *(const uint4*)(stg + (r * 32 + px) * PIXB + ((lc ^ (px & 7)) << 4));
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
                const uint32_t m = 0u - (kw[j / JPR] >> ((j % JPR) * PPJ + lcol) & 1u);
                o.x &= m; o.y &= m; o.z &= m; o.w &= m;
            }
            const i32x4 v = {(int)o.x, (int)o.y, (int)o.z, (int)o.w};
            __builtin_amdgcn_raw_buffer_store_b128(v, rout, out_off(j, ln, y0, x0), 0, ST_THROUGH);
            if constexpr (SKIP) __builtin_amdgcn_sched_barrier(0);
        }
        // A second look, where the first one was too early: the patch is requested now, or in the next phase.
        if (!early && !none) {
            if (wave == 0) {
                const bool ready = __builtin_amdgcn_ballot_w64(again >= (uint32_t)nu.layer) == ~0ull;
                if (lane == 0) __hip_atomic_store(&s_again[team], (uint32_t)turn * 2 + 2 + ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            uint32_t v;
            while ((v = __builtin_amdgcn_readfirstlane(__hip_atomic_load(&s_again[team], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))) >> 1 != (uint32_t)turn + 1) {}
            fetch = v & 1;
            __builtin_amdgcn_sched_barrier(0);
            if (fetch) {
                __amdgpu_buffer_rsrc_t rnow = rsrc_of(layer_in(nu.layer), nu.n, true);
#pragma unroll
                for (int j = 0; j < NPRE; ++j) load_piece(j, tt, rnow, nu.y0, nu.x0);
                asm volatile("s_waitcnt vmcnt(%0)" :: "n"(NPRE) : "memory");      // the stores, not the patch behind them
                mark_done(cur);
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                mark_done(cur);
            }
            lds_dma_wait();                                  // the compiler need not wait for more than an early patch below
        }
        }
        const bool told = !early && !none;
        prev = cur; cur = nu; ++turn;
        if (!told) {
            if (at_end || none || !__builtin_amdgcn_readfirstlane(ready0)) {      // somebody may wait for this unit: the team beside this one included
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                mark_done(prev);
                if (at_end) return true;
                word_due = false;
            } else word_due = true;
        } else word_due = false;
        resident = front_layer;
        body_barrier();                                      // 1
        if (fetch) { int tt = ttid; asm volatile("" : "+v"(tt)); store_patch(tt); }
        loaded = fetch;
        if (cur.layer < a.layers && cur.layer != bias_layer) { store_bias(load_bias(cur.layer)); bias_layer = cur.layer; }
        body_barrier();                                      // 2
        return false;
    };

    if (team == 1) { body_barrier(); resident = 0; body_barrier(); }      // the first unit is the other team's
    auto run = [&](auto few_c) __attribute__((always_inline)) {
    for (;;) {
        if (word_due && (cur.layer >= a.layers || !loaded)) {        // ahead of any wait
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            mark_done(prev);
            word_due = false;
        }
        if (cur.layer >= a.layers) break;
        if (!loaded || cur.layer != resident) {
            if (cur.layer != resident) {
                int w = wave;
                asm volatile("" : "+s"(w));                  // as `lane`: its 18 offsets are not kept
                lds_dma<256, WBYTES>(lds_w, a.wp + (size_t)cur.layer * (WBYTES / 16), w, lane_now());
            }
            float bias = load_bias(cur.layer);
            if (!loaded) {
                int tt = ttid;
                asm volatile("" : "+v"(tt));
                int polls = 0;                               // every wave for itself
                while (__builtin_amdgcn_ballot_w64(load_words(cur) >= (uint32_t)cur.layer) != ~0ull) {
                    if (lost() || ++polls > BODY_POLLS) {
                        __hip_atomic_store(&s_lost, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                        tell_host();
                        break;
                    }
                }
                // Marks the result where no ReLU drops it.
                if (lost()) bias = __builtin_nanf("");
                __amdgpu_buffer_rsrc_t rin = rsrc_of(layer_in(cur.layer), cur.n, true);
#pragma unroll
                for (int j = 0; j < NPRE; ++j) load_piece(j, tt, rin, cur.y0, cur.x0);
                store_patch(tt);
            }
            store_bias(bias); bias_layer = cur.layer;
            lds_dma_wait();
            team_sync();
        }
        resident = cur.layer;
        if (layer_skips(cur.layer) ? unit(std::integral_constant<bool, true>{}, few_c) : unit(std::integral_constant<bool, false>{}, few_c)) break;
    }
    };
    if (layer_units <= FEW_UNITS * (int)gridDim.x) run(std::integral_constant<bool, true>{});
    else run(std::integral_constant<bool, false>{});
}

bool rh_conv_body_pairs(int n_cu, int N, int H, int W) { return body_pair_rows(N, H, W, n_cu) > 0; }

hipError_t rh_launch_conv_body(hipStream_t stream, int device, int n_cu, body_args a)
{
    constexpr int lds = BODY_PAIR_LDS(BODY_PAIR_MOST);
    static_assert(lds >= BODY_PAIR_LDS(16) && lds >= 9 * 64 * 64 * 2 + 2 * 10 * PW * 128, "the largest of them");
    static bool attr_done[RH_MAX_DEVICES] = {};            // the attribute is per device
    if (!attr_done[device]) {
        hipError_t e = hipFuncSetAttribute((const void*)k_conv_mfma_body<false>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e == hipSuccess) e = hipFuncSetAttribute((const void*)k_conv_mfma_body<true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_done[device] = true;
    }
    const long long cells_x = (a.W + 31) / 32, cells_img = cells_x * ((a.H + 7) / 8), units = a.N * cells_img;
    if (units * cells_img >= 1ll << 32) return hipErrorInvalidValue;
    a.img_magic = (uint32_t)(0xFFFFFFFFu / cells_img + 1);   // x / d = high word of x * magic for x * d < 2^32; 0: d = 1
    a.row_magic = (uint32_t)(0xFFFFFFFFu / cells_x + 1);
    const long long most = body_pair_units(a.N, a.H, a.W, 4);      // at least as many as half tiles
    const int grid = (int)(most < n_cu ? most : n_cu);
    if (a.keep) hipLaunchKernelGGL(k_conv_mfma_body<true>, dim3(grid), dim3(512), lds, stream, a);
    else hipLaunchKernelGGL(k_conv_mfma_body<false>, dim3(grid), dim3(512), lds, stream, a);
    return hipGetLastError();
}
