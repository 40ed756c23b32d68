// Cross-stream macroblock selection (Sec. 3.3.1): the top-k of each segment's importance
// queue, or a threshold, as an exact k-th-key radix select plus an ordered ballot/prefix-sum
// compaction.  No sort of the queue is materialised: a macroblock is selected iff its key is
// above the k-th key, or equals it and is among the first `budget` such macroblocks in
// ascending flat index.
#include <string.h>

#include "rh_internal.h"

// Order-preserving image of an fp32 importance: larger key = more important.
// -0 is treated as +0 and every NaN maps to 0, below all numbers (-inf maps to 0x007FFFFF).
__device__ __forceinline__ uint32_t imp_key(float v)
{
    uint32_t b = __float_as_uint(v);
    if ((b & 0x7FFFFFFFu) > 0x7F800000u) return 0u;
    if (b == 0x80000000u) b = 0u;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Kernel 1: one workgroup per segment.  Finds the segment's threshold key T and tie budget,
// then the number of selected macroblocks and admitted ties of each of its frames.
// seg_par[seg] = {g_begin, g_end, k, thr bits}.
// A queue of up to KREG * 1024 keys (a 30-frame chunk of 480x272 streams is 15k) is read from
// global memory once and kept in registers over the three radix passes; a longer one is read anew for each
// pass, eight loads in flight per thread.  (64 keys per thread cost 128 registers and spills: slower at every size.)
#define KREG 16
#define BINS 2048            // digits of 11, 11 and 10 bits
// Segment tables travel as kernel arguments (copied at launch), so the caller's array may be
// freed as soon as rh_select_regions returns and no host synchronisation is needed.
struct seg_chunk { uint32_t n, first; uint32_t fb[64], fe[64], k[64], thr[64]; };

#define FCHUNK 1024          // frames whose counts are held in LDS at a time

// Inclusive prefix sum over the wave, by DPP
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v)
{
#define STEP(ctrl, rows) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xF, false)
    STEP(0x111 /* row_shr:1 */, 0xF); STEP(0x112, 0xF); STEP(0x114, 0xF); STEP(0x118, 0xF);
    STEP(0x142 /* row_bcast:15 */, 0xA); STEP(0x143 /* row_bcast:31 */, 0xC);
#undef STEP
    return v;
}

// The bin of `hist` that holds the k-th key (k = remaining, counted from the top) goes to *s_prefix behind the digits that are
// known, and what is left of k to *s_remaining.  All 1024 threads, which have counted; they find both after it.
__device__ __forceinline__ void pick_bin(const uint32_t* hist, int shift, uint32_t prefix, uint32_t remaining, uint32_t* s_wtot,
                                         uint32_t* s_prefix, uint32_t* s_remaining)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // bin t holds the k-th key iff  above(t) < remaining <= above(t) + hist[t],  above(t) = sum of
    // the bins over t.  Thread t holds the bins 2047 - 2t and 2046 - 2t, so that is a prefix sum.
    const uint32_t b1 = BINS - 1 - 2 * tid, h1 = hist[b1], h0 = hist[b1 - 1], incl = wave_prefix(h1 + h0);
    if (lane == 63) s_wtot[wave] = incl;
    __syncthreads();
    const uint32_t tot = wave_prefix(s_wtot[lane & 15]);           // lanes 0..15: inclusive sums of the waves' totals
    const uint32_t above1 = incl - h1 - h0 + (wave ? (uint32_t)__builtin_amdgcn_readlane((int)tot, __builtin_amdgcn_readfirstlane(wave ? wave - 1 : 0)) : 0u);
    const uint32_t above0 = above1 + h1;
    if (above1 < remaining && remaining <= above1 + h1) { *s_prefix = prefix | (b1 << shift); *s_remaining = remaining - above1; }
    if (above0 < remaining && remaining <= above0 + h0) { *s_prefix = prefix | ((b1 - 1) << shift); *s_remaining = remaining - above0; }
    __syncthreads();
}

// The whole top-k selection in one launch, where every segment's queue stays in one workgroup's registers.  A segment
// selects min(k, n) keys, so where its part of the list begins is known without the other segments' keys; ties go
// to the smallest indexes, so one prefix sum over the queue numbers them and what is selected, and frames need no counts.
// Two launches / this one, us of kernels: one segment of 240 keys 11.6 / 6.8, of 8160 behind a step of convs 27.9 / 17.1.
__global__ __launch_bounds__(1024) void k_select_once(seg_chunk c, int F, const float* __restrict__ imp, int per, uint8_t* __restrict__ mask,
                                                      uint32_t* __restrict__ list, uint32_t* __restrict__ n_sel)
{
    __shared__ uint32_t hist[BINS];
    __shared__ uint32_t s_wtot[16];
    __shared__ uint32_t s_prefix, s_remaining;
    __shared__ __attribute__((aligned(16))) uint32_t s_cnt[KREG * 16];     // keys above the threshold | ties << 16 of a wave's 64 keys
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), seg = blockIdx.x;
    const uint32_t g0 = c.fb[seg] * (uint32_t)per, n = c.fe[seg] * (uint32_t)per - g0, k = min(c.k[seg], n);
    uint32_t keys[KREG];
#pragma unroll
    for (int j = 0; j < KREG; ++j) {
        const uint32_t i = (uint32_t)j * 1024u + tid;
        keys[j] = i < n ? imp_key(imp[g0 + i]) : 0u;
    }
    // frames of no segment in front of this one, and behind the last
    for (uint32_t i = (seg ? c.fe[seg - 1] * (uint32_t)per : 0u) + tid; i < g0; i += 1024) mask[i] = 0;
    if (seg + 1 == (int)c.n) for (uint32_t i = g0 + n + tid; i < (uint32_t)F * (uint32_t)per; i += 1024) mask[i] = 0;
    const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)wave_prefix(lane < seg ? min(c.k[lane], (c.fe[lane] - c.fb[lane]) * (uint32_t)per) : 0u), 63);
    if (seg + 1 == (int)c.n && tid == 0) *n_sel = first + k;
    uint32_t T = 0xFFFFFFFFu, budget = 0;                      // no key reaches 0xFFFFFFFF
    if (k) {
        uint32_t prefix = 0, remaining = k;
        for (int pass = 0; pass < 3; ++pass) {
            const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
            const uint32_t digit = pass == 2 ? 1023u : 2047u, hi_mask = pass == 0 ? 0u : (0xFFFFFFFFu << (pass == 1 ? 21 : 10));
            hist[tid] = 0; hist[tid + 1024] = 0;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < KREG; ++j) {
                const uint32_t i = (uint32_t)j * 1024u + tid;
                if (i < n && (keys[j] & hi_mask) == prefix) atomicAdd(&hist[keys[j] >> shift & digit], 1u);
            }
            __syncthreads();
            pick_bin(hist, shift, prefix, remaining, s_wtot, &s_prefix, &s_remaining);
            prefix = s_prefix; remaining = s_remaining;
        }
        T = prefix; budget = remaining;
    }
#pragma unroll
    for (int j = 0; j < KREG; ++j) {
        const bool in = (uint32_t)j * 1024u + tid < n;
        const uint32_t gt = (uint32_t)__popcll(__ballot(in && keys[j] > T)), eq = (uint32_t)__popcll(__ballot(in && keys[j] == T));
        if (lane == 0) s_cnt[j * 16 + wave] = gt | eq << 16;
    }
    __syncthreads();
    // every wave sums up all 256 counts in order of the keys: lane l has four of them, from wave l % 4 * 4 of row l / 4 on
    static_assert(KREG == 16, "four counts a lane");
    const uint4 v = ((const uint4*)s_cnt)[lane];
    const uint32_t x0 = wave_prefix(v.x + v.y + v.z + v.w) - (v.x + v.y + v.z + v.w), x1 = x0 + v.x, x2 = x1 + v.y, x3 = x2 + v.z;
    const uint32_t before = (wave & 3) == 0 ? x0 : (wave & 3) == 1 ? x1 : (wave & 3) == 2 ? x2 : x3;
    const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
    for (int j = 0; j < KREG; ++j) {
        const uint32_t i = (uint32_t)j * 1024u + tid;
        if ((uint32_t)j * 1024u >= n) break;                   // uniform over the workgroup
        const bool gt = i < n && keys[j] > T, eq = i < n && keys[j] == T;
        const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)before, j * 4 + (wave >> 2));
        const uint32_t ties = (b >> 16) + (uint32_t)__popcll(__ballot(eq) & below);
        const uint32_t at = first + (b & 0xFFFFu) + (uint32_t)__popcll(__ballot(gt) & below) + min(ties, budget);
        const bool sel = gt || (eq && ties < budget);
        if (i < n) mask[g0 + i] = sel ? 1 : 0;
        if (sel) list[at] = g0 + i;
    }
}

// INLINE: the call's segments are all in c (seg_par is not read), and the frames without a segment get their
// counts (0) here; otherwise k_upload_segments has written seg_par and frame_seg.
template <bool INLINE>
__global__ __launch_bounds__(1024) void k_select_kth(seg_chunk c, int F, const float* __restrict__ imp,
                                                     const uint32_t* __restrict__ seg_par, int mode,
                                                     int per, uint32_t* __restrict__ seg_T,
                                                     uint32_t* __restrict__ frame_nsel,
                                                     uint32_t* __restrict__ frame_ties)
{
    __shared__ uint32_t hist[BINS];
    __shared__ uint32_t s_wtot[16];
    __shared__ uint32_t s_prefix, s_remaining;
    __shared__ uint32_t s_gt[FCHUNK], s_eq[FCHUNK], s_scan[2][FCHUNK];
    const int tid = threadIdx.x, seg = blockIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const uint32_t g0 = INLINE ? c.fb[seg] * (uint32_t)per : seg_par[4 * seg], g1 = INLINE ? c.fe[seg] * (uint32_t)per : seg_par[4 * seg + 1];
    if (INLINE) {
        for (uint32_t f = (seg ? c.fe[seg - 1] : 0u) + tid; f < c.fb[seg]; f += 1024) frame_nsel[f] = 0;
        if (seg + 1 == (int)c.n) for (uint32_t f = c.fe[seg] + tid; f < (uint32_t)F; f += 1024) frame_nsel[f] = 0;
    }
    const uint32_t n = g1 - g0;
    const uint32_t f0 = g0 / per, f1 = g1 / per;
    uint32_t k = INLINE ? c.k[seg] : seg_par[4 * seg + 2];
    // a queue that fits is read once and stays in registers for the radix passes and the counts
    const bool in_regs = n <= KREG * 1024u && f1 - f0 <= FCHUNK;
    uint32_t keys[KREG];
    if (in_regs) {
#pragma unroll
        for (int j = 0; j < KREG; ++j) {
            const uint32_t i = (uint32_t)j * 1024u + tid;
            keys[j] = i < n ? imp_key(imp[g0 + i]) : 0u;
        }
    }
    uint32_t T, budget;
    if (mode == RH_THRESHOLD) {
        float thr = __uint_as_float(INLINE ? c.thr[seg] : seg_par[4 * seg + 3]);
        if (thr != thr) { T = 0xFFFFFFFFu; budget = 0u; }       // NaN threshold selects nothing
        else { T = imp_key(thr); budget = 0xFFFFFFFFu; }         // every key == T is taken
    } else {
        if (k > n) k = n;
        if (k == 0) { T = 0xFFFFFFFFu; budget = 0u; }            // no key reaches 0xFFFFFFFF
        else {
            uint32_t prefix = 0, remaining = k;
            for (int pass = 0; pass < 3; ++pass) {
                const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
                const uint32_t digit = pass == 2 ? 1023u : 2047u, hi_mask = pass == 0 ? 0u : (0xFFFFFFFFu << (pass == 1 ? 21 : 10));
                hist[tid] = 0; hist[tid + 1024] = 0;
                __syncthreads();
                if (in_regs) {
#pragma unroll
                    for (int j = 0; j < KREG; ++j) {
                        const uint32_t i = (uint32_t)j * 1024u + tid;
                        if (i < n && (keys[j] & hi_mask) == prefix) atomicAdd(&hist[keys[j] >> shift & digit], 1u);
                    }
                } else {
                    for (uint32_t i0 = 0; i0 < n; i0 += 8 * 1024) {
                        float v[8];
#pragma unroll
                        for (int u = 0; u < 8; ++u) { const uint32_t i = i0 + u * 1024 + tid; v[u] = imp[g0 + min(i, n - 1u)]; }
#pragma unroll
                        for (int u = 0; u < 8; ++u) {
                            const uint32_t i = i0 + u * 1024 + tid, key = imp_key(v[u]);
                            if (i < n && (key & hi_mask) == prefix) atomicAdd(&hist[key >> shift & digit], 1u);
                        }
                    }
                }
                __syncthreads();
                pick_bin(hist, shift, prefix, remaining, s_wtot, &s_prefix, &s_remaining);
                prefix = s_prefix; remaining = s_remaining;
            }
            T = prefix; budget = remaining;
        }
    }
    if (tid == 0) seg_T[seg] = T;
    // per-frame counts of keys above T (gt) and equal to T (eq); the ties are then dealt to the
    // frames in ascending order: a frame may take  min(eq, budget - ties of the frames before it)
    uint32_t left = budget;                                    // uniform over the workgroup
    for (uint32_t c0 = f0; c0 < f1; c0 += FCHUNK) {
        const uint32_t nf = (f1 - c0) < FCHUNK ? (f1 - c0) : FCHUNK;
        if (in_regs) {                                         // one chunk: counts straight from the registers
            if ((uint32_t)tid < nf) { s_gt[tid] = 0; s_eq[tid] = 0; }
            __syncthreads();
#pragma unroll
            for (int j = 0; j < KREG; ++j) {
                if ((uint32_t)j * 1024u >= n) break;               // uniform over the workgroup
                const uint32_t i = (uint32_t)j * 1024u + tid;
                const bool gt = i < n && keys[j] > T, eq = i < n && keys[j] == T;
                const uint32_t fr = i / (uint32_t)per;             // frame within the segment
                unsigned long long act = __ballot(gt || eq);
                while (act) {                                      // one round per frame present in the wave
                    const int first = __ffsll((long long)act) - 1;
                    const uint32_t fs = (uint32_t)__builtin_amdgcn_readlane((int)fr, first);
                    const unsigned long long mg = __ballot(gt && fr == fs), me = __ballot(eq && fr == fs);
                    const uint32_t ng = (uint32_t)__popcll(mg), ne = (uint32_t)__popcll(me);
                    if (lane == first) { if (ng) atomicAdd(&s_gt[fs], ng); if (ne) atomicAdd(&s_eq[fs], ne); }
                    act &= ~(mg | me);
                }
            }
        } else {                                               // one wave per frame, from global memory
            for (uint32_t j = wave; j < nf; j += 16) {
                const size_t fb = (size_t)(c0 + j) * per;
                uint32_t gt = 0, eq = 0;
                for (int i = lane; i < per; i += 64) {
                    const uint32_t key = imp_key(imp[fb + i]);
                    gt += key > T; eq += key == T;
                }
                for (int o = 32; o > 0; o >>= 1) { gt += __shfl_xor(gt, o); eq += __shfl_xor(eq, o); }
                if (lane == 0) { s_gt[j] = gt; s_eq[j] = eq; }
            }
        }
        __syncthreads();
        // inclusive scan of eq over the chunk
        int cur = 0;
        if ((uint32_t)tid < nf) s_scan[0][tid] = s_eq[tid];
        __syncthreads();
        for (uint32_t d = 1; d < nf; d <<= 1) {
            if ((uint32_t)tid < nf) {
                uint32_t v = s_scan[cur][tid];
                if ((uint32_t)tid >= d) v += s_scan[cur][tid - d];    // at most n < 2^32 in total: no overflow
                s_scan[cur ^ 1][tid] = v;
            }
            cur ^= 1;
            __syncthreads();
        }
        if ((uint32_t)tid < nf) {
            const uint32_t eq = s_eq[tid], before = s_scan[cur][tid] - eq;
            const uint32_t room = before < left ? left - before : 0u;
            const uint32_t ties = eq < room ? eq : room;
            frame_nsel[c0 + tid] = s_gt[tid] + ties; frame_ties[c0 + tid] = ties;
        }
        const uint32_t tot = s_scan[cur][nf - 1];
        left = tot < left ? left - tot : 0u;
        __syncthreads();
    }
}

// Exclusive prefix count of a predicate over a 256-thread workgroup, in thread order.
__device__ __forceinline__ uint32_t block_prefix256(bool pred, uint32_t* s_w /*[4]*/, uint32_t& total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    unsigned long long m = __ballot(pred);
    uint32_t pre = __popcll(m & ((1ull << lane) - 1ull));
    __syncthreads();                       // s_w free for reuse
    if (lane == 0) s_w[w] = __popcll(m);
    __syncthreads();
    uint32_t off = 0; total = 0;
    for (int i = 0; i < 4; ++i) { uint32_t c = s_w[i]; if (i < w) off += c; total += c; }
    return pre + off;
}

// Kernel 2: one workgroup per frame writes the frame's mask and its slice of the list.
template <bool INLINE>
__global__ __launch_bounds__(256) void k_select_write(seg_chunk c, const float* __restrict__ imp,
                                                      const int32_t* __restrict__ frame_seg,
                                                      const uint32_t* __restrict__ seg_T,
                                                      const uint32_t* __restrict__ frame_nsel,
                                                      const uint32_t* __restrict__ frame_ties,
                                                      int per, int F, uint8_t* __restrict__ mask,
                                                      uint32_t* __restrict__ list,
                                                      uint32_t* __restrict__ n_sel)
{
    __shared__ uint32_t s_w[4];
    __shared__ uint32_t s_base;
    const int tid = threadIdx.x, f = blockIdx.x;
    if (tid == 0) s_base = 0;
    __syncthreads();
    uint32_t local = 0;
    if (!INLINE || c.n)                    // no segment at all: no counts
        for (int i = tid; i < f; i += 256) if (INLINE || frame_seg[i] >= 0) local += frame_nsel[i];
    if (local) atomicAdd(&s_base, local);
    __syncthreads();
    const uint32_t base = s_base;
    int seg = -1;
    if constexpr (INLINE) {
        const int s = tid & 63;            // lane s looks at segment s
        const unsigned long long m = __ballot(s < (int)c.n && c.fb[s] <= (uint32_t)f && (uint32_t)f < c.fe[s]);
        if (m) seg = __ffsll((long long)m) - 1;
    } else seg = frame_seg[f];
    const size_t fb = (size_t)f * per;
    if (seg < 0) {
        for (int i = tid; i < per; i += 256) mask[fb + i] = 0;
        if (f == F - 1 && tid == 0) *n_sel = base;
        return;
    }
    const uint32_t T = seg_T[seg], ties_allowed = frame_ties[f];
    uint32_t run_sel = 0, run_eq = 0;
    for (int p0 = 0; p0 < per; p0 += 256) {
        const int i = p0 + tid;
        const bool valid = i < per;
        const uint32_t key = valid ? imp_key(imp[fb + i]) : 0u;
        const bool gt = valid && key > T, eq = valid && key == T;
        uint32_t tot_eq, tot_sel;
        uint32_t eq_pre = block_prefix256(eq, s_w, tot_eq);
        const bool sel = gt || (eq && (run_eq + eq_pre) < ties_allowed);
        uint32_t sel_pre = block_prefix256(sel, s_w, tot_sel);
        if (valid) {
            mask[fb + i] = sel ? 1 : 0;
            if (sel) list[base + run_sel + sel_pre] = (uint32_t)(fb + i);
        }
        run_eq += tot_eq; run_sel += tot_sel;
    }
    if (f == F - 1 && tid == 0) *n_sel = base + run_sel;
}

// One workgroup.  The first chunk of a call (c.first == 0) also marks every frame as belonging to
// no segment before the segments' frames are labelled.
__global__ __launch_bounds__(256) void k_upload_segments(seg_chunk c, int per, int F, uint32_t* __restrict__ seg_par,
                                                         int32_t* __restrict__ frame_seg)
{
    if (c.first == 0) {
        for (int f = threadIdx.x; f < F; f += 256) frame_seg[f] = -1;
        __syncthreads();
    }
    for (uint32_t s = 0; s < c.n; ++s) {
        if (threadIdx.x == 0) {
            uint32_t* p = seg_par + 4 * (size_t)(c.first + s);
            p[0] = c.fb[s] * (uint32_t)per; p[1] = c.fe[s] * (uint32_t)per; p[2] = c.k[s]; p[3] = c.thr[s];
        }
        for (uint32_t f = c.fb[s] + threadIdx.x; f < c.fe[s]; f += 256) frame_seg[f] = (int32_t)(c.first + s);
    }
}

// k_select_once: queues that stay in registers, and few enough macroblocks outside the segments for one workgroup to clear
static bool in_one_launch(const rh_segment* segs, int nseg, int mode, int F, int per)
{
    if (mode != RH_TOPK || nseg < 1 || nseg > 64) return false;
    uint32_t longest = 0, covered = 0;                       // frames
    for (int i = 0; i < nseg; ++i) {
        const uint32_t len = segs[i].frame_end - segs[i].frame_begin;
        longest = longest > len ? longest : len; covered += len;
    }
    return (uint64_t)longest * (uint64_t)per <= KREG * 1024u && (uint64_t)((uint32_t)F - covered) * (uint64_t)per <= 65536u;
}

hipError_t rh_enqueue_select(hipStream_t stream, const rh_select_scratch& sc, const float* imp, int F, int per,
                                 const rh_segment* segs, int nseg, int mode, uint8_t* mask, uint32_t* list, uint32_t* n_sel)
{
    seg_chunk c;
    auto fill = [&](int s0) {
        c.n = (uint32_t)((nseg - s0) < 64 ? (nseg - s0) : 64); c.first = (uint32_t)s0;
        for (uint32_t i = 0; i < c.n; ++i) {
            const rh_segment& g = segs[s0 + i];
            c.fb[i] = g.frame_begin; c.fe[i] = g.frame_end; c.k[i] = g.k; memcpy(&c.thr[i], &g.thr, 4);
        }
    };
    if (in_one_launch(segs, nseg, mode, F, per)) {
        fill(0);
        hipLaunchKernelGGL(k_select_once, dim3(nseg), dim3(1024), 0, stream, c, F, imp, per, mask, list, n_sel);
        return hipGetLastError();
    }
    if (nseg <= 64) {                                        // one launch less: 5 us with its gap
        fill(0);
        if (nseg > 0)
            hipLaunchKernelGGL(k_select_kth<true>, dim3(nseg), dim3(1024), 0, stream, c, F, imp, sc.seg_par, mode, per, sc.seg_T,
                               sc.frame_nsel, sc.frame_ties);
        hipLaunchKernelGGL(k_select_write<true>, dim3(F), dim3(256), 0, stream, c, imp, sc.frame_seg, sc.seg_T, sc.frame_nsel,
                           sc.frame_ties, per, F, mask, list, n_sel);
        return hipGetLastError();
    }
    for (int s0 = 0; s0 < nseg; s0 += 64) {
        fill(s0);
        hipLaunchKernelGGL(k_upload_segments, dim3(1), dim3(256), 0, stream, c, per, F, sc.seg_par, sc.frame_seg);
    }
    hipLaunchKernelGGL(k_select_kth<false>, dim3(nseg), dim3(1024), 0, stream, c, F, imp, sc.seg_par, mode, per, sc.seg_T,
                       sc.frame_nsel, sc.frame_ties);
    hipLaunchKernelGGL(k_select_write<false>, dim3(F), dim3(256), 0, stream, c, imp, sc.frame_seg, sc.seg_T, sc.frame_nsel,
                       sc.frame_ties, per, F, mask, list, n_sel);
    return hipGetLastError();
}

// Argument checks shared by both entry points; returns a message or null.
const char* rh_check_select_args(const float* importance, int F, const rh_segment* segs, int nseg, int mode,
                                     const uint8_t* mask, const uint32_t* list, const uint32_t* n_sel, rh_status* st)
{
    *st = RH_E_INVALID;
    if (!importance || !mask || !list || !n_sel || (nseg > 0 && !segs) || nseg < 0) return "null argument";
    if (mode != RH_TOPK && mode != RH_THRESHOLD) return "bad mode";
    if (nseg > F) return "more segments than frames";
    uint32_t prev_end = 0;
    for (int s = 0; s < nseg; ++s) {
        const rh_segment& g = segs[s];
        if (g.frame_begin > g.frame_end || g.frame_end > (uint32_t)F || g.frame_begin < prev_end)
            return "a segment is out of range, unordered or overlapping";
        prev_end = g.frame_end;
    }
    *st = RH_OK;
    return nullptr;
}

rh_status rh_launch_select(rh_ctx* ctx, const float* imp, int F, const rh_segment* segs, int nseg, int mode,
                           uint8_t* mask, uint32_t* list, uint32_t* n_sel)
{
    rh_status st;
    if (const char* msg = rh_check_select_args(imp, F, segs, nseg, mode, mask, list, n_sel, &st))
        RH_FAIL(ctx, st, "rh_select_regions: %s", msg);
    const int n_up = nseg > 64 ? (nseg + 63) / 64 : 0, once = in_one_launch(segs, nseg, mode, F, ctx->per);
    rh_prof_scope ps(ctx, RH_PROF_SELECT, once ? 1 : n_up + (nseg > 0 ? 2 : 1));
    const rh_select_scratch sc = {ctx->frame_seg, ctx->seg_par, ctx->seg_T, ctx->frame_nsel, ctx->frame_ties};
    RH_HIP(ctx, rh_enqueue_select(ctx->stream, sc, imp, F, ctx->per, segs, nseg, mode, mask, list, n_sel));
    return RH_OK;
}

