// Region-aware bin packing (Alg. 1) on macroblock indexes, entirely on the GPU:
//   k_plan_regions / k_plan_label : RegionProps + Bound + Partition, one wave per frame (rows as 64-bit masks), or for
//                  larger frames one workgroup (labels in LDS)
//   k_plan_rank  : Sort by importance density (rank by counting; the order is total)
//   k_plan_place : the serial first-fit over the ordered free-rectangle list, one wave,
//                  lanes test free rectangles in parallel, the list lives in registers
//   k_plan_emit  : placement rows for boxes and macroblocks
//   k_plan_fused : all of these in one launch, for batches of few frames
#include "rh_internal.h"

#define NONE 0xFFFFFFFFu

// One workgroup per frame.  LDS: lab[per], cminx[per], cmaxx[per], cmaxy[per] and, when it fits
// (imp_in_lds), the frame's importance values: a box leader adds up to T*T of them one after the
// other in a fixed order, which from global memory is a chain of that many load latencies.
// A region's label is the smallest in-frame index of its macroblocks.
__global__ __launch_bounds__(256) void k_plan_label(const uint8_t* __restrict__ mask,
                                                    const float* __restrict__ imp, int mbw, int mbh,
                                                    int conn, int T, int sort_policy, int imp_in_lds,
                                                    uint32_t* __restrict__ owner_id,
                                                    rh_rawbox* __restrict__ raw, uint32_t* pcount)
{
    extern __shared__ uint32_t sm[];
    const int per = mbw * mbh, tid = threadIdx.x, f = blockIdx.x;
    volatile uint32_t* lab = sm;
    uint32_t* cminx = sm + per; uint32_t* cmaxx = sm + 2 * per; uint32_t* cmaxy = sm + 3 * per;
    float* simp = (float*)(sm + 4 * per);
    __shared__ int s_changed;
    const size_t base = (size_t)f * per;
    for (int i = tid; i < per; i += 256) {
        lab[i] = mask[base + i] ? (uint32_t)i : NONE;
        cminx[i] = NONE; cmaxx[i] = 0; cmaxy[i] = 0;
        if (imp_in_lds) simp[i] = imp[base + i];
    }
    // RegionProps: iterate "take the smallest label around me, then follow it to its root"
    // until nothing changes.  Labels only decrease and always name a macroblock of the same
    // region, so the fixed point is the region's smallest index everywhere.
    for (;;) {
        __syncthreads();
        if (tid == 0) s_changed = 0;
        __syncthreads();
        int any = 0;
        for (int i = tid; i < per; i += 256) {
            uint32_t cur = lab[i];
            if (cur == NONE) continue;
            const int y = i / mbw, x = i - y * mbw;
            uint32_t m = cur;
            for (int dy = -1; dy <= 1; ++dy) {
                const int ny = y + dy;
                if (ny < 0 || ny >= mbh) continue;
                for (int dx = -1; dx <= 1; ++dx) {
                    if ((dx == 0 && dy == 0) || (conn == 4 && dx != 0 && dy != 0)) continue;
                    const int nx = x + dx;
                    if (nx < 0 || nx >= mbw) continue;
                    uint32_t ln = lab[ny * mbw + nx];
                    m = ln < m ? ln : m;
                }
            }
            for (uint32_t r = lab[m]; r < m; r = lab[m]) m = r;
            if (m < cur) { lab[i] = m; any = 1; }
        }
        if (any) s_changed = 1;
        __syncthreads();
        if (!s_changed) break;
    }
    // Bound: bounding box of every region, kept at the root's slot (min y is the root's row).
    for (int i = tid; i < per; i += 256) {
        uint32_t r = lab[i];
        if (r == NONE) continue;
        const int y = i / mbw, x = i - y * mbw;
        atomicMin(&cminx[r], (uint32_t)x); atomicMax(&cmaxx[r], (uint32_t)x); atomicMax(&cmaxy[r], (uint32_t)y);
    }
    __syncthreads();
    // Partition: the region's bounding box is cut on a T x T grid anchored at its top-left.
    // Every macroblock looks through its own cell in raster order: the first macroblock of
    // the same region there leads the box and describes it.
    for (int i = tid; i < per; i += 256) {
        uint32_t r = lab[i];
        if (r == NONE) continue;
        const int y = i / mbw, x = i - y * mbw;
        const int ry = r / mbw, minx = cminx[r], maxx = cmaxx[r], maxy = cmaxy[r];
        const int wx0 = minx + ((x - minx) / T) * T, wy0 = ry + ((y - ry) / T) * T;
        const int wx1 = min(wx0 + T - 1, maxx), wy1 = min(wy0 + T - 1, maxy);
        int leader = -1, x0 = 1 << 30, x1 = -1, y0 = 1 << 30, y1 = -1;
        float sum = 0.0f;
        for (int yy = wy0; yy <= wy1; ++yy) {
            for (int xx = wx0; xx <= wx1; ++xx) {
                const int j = yy * mbw + xx;
                if (lab[j] != r) continue;
                if (leader < 0) leader = j;
                if (leader != i) break;                      // only the leader needs the rest
                sum = __fadd_rn(sum, imp_in_lds ? simp[j] : imp[base + j]);   // fp32, ascending flat index
                x0 = min(x0, xx); x1 = max(x1, xx); y0 = min(y0, yy); y1 = max(y1, yy);
            }
            if (leader >= 0 && leader != i) break;
        }
        owner_id[base + i] = (uint32_t)(base + leader);
        if (leader == i) {
            uint32_t slot = atomicAdd(&pcount[3], 1u);
            rh_rawbox b;
            b.frame = f; b.mbx0 = x0; b.mby0 = y0; b.wmb = x1 - x0 + 1; b.hmb = y1 - y0 + 1;
            b.id = (uint32_t)(base + i); b.sum = sum;
            const int area = (x1 - x0 + 1) * (y1 - y0 + 1);
            b.key = sort_policy == RH_SORT_AREA ? (double)area : (double)sum / (double)area;
            raw[slot] = b;
        }
    }
}

// Orders the LDS accesses of one wave: what lanes wrote before it is what any lane reads after it.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The packing order on integers: a larger ord_key comes first, equal keys go by ascending id.  Same
// order as box_before: doubles map to their order-preserving 64-bit image (-0 = +0), NaN to 0 (last;
// no finite key or -inf maps that low: -inf gives 0x000FFFFFFFFFFFFF).
__device__ __forceinline__ unsigned long long ord_key(double k)
{
    if (k != k) return 0ull;
    unsigned long long b = (unsigned long long)__double_as_longlong(k);
    if (b == 0x8000000000000000ull) b = 0ull;
    return (b & 0x8000000000000000ull) ? ~b : (b | 0x8000000000000000ull);
}

// a before b in the packing order: higher key (density, or area) first, NaN last, ties by ascending id.
__device__ __forceinline__ bool box_before(double ka, uint32_t ia, double kb, uint32_t ib)
{
    const bool an = ka != ka, bn = kb != kb;
    if (an != bn) return bn;
    if (!an) { if (ka > kb) return true; if (ka < kb) return false; }
    return ia < ib;
}

// Sort by counting: the rank of a box is the number of boxes before it.  A wave ranks RANK_PER boxes at a
// time, its lanes compare them with 64 others each step; keys pass through LDS in tiles.  (A thread per
// box took 87 us for 752 boxes, three workgroups going through all boxes one by one.)
#define RANK_PER 4
#define RANK_TILE 1024

__global__ __launch_bounds__(256) void k_plan_rank(const rh_rawbox* __restrict__ raw,
                                                   const uint32_t* __restrict__ pcount,
                                                   rh_rawbox* __restrict__ sorted,
                                                   uint32_t* __restrict__ rank_of_id)
{
    __shared__ unsigned long long s_key[RANK_TILE];
    __shared__ uint32_t s_id[RANK_TILE];
    const uint32_t n = pcount[3];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (uint32_t b0 = blockIdx.x * (4 * RANK_PER); b0 < n; b0 += gridDim.x * (4 * RANK_PER)) {       // uniform over the workgroup
        const uint32_t i0 = b0 + wave * RANK_PER;
        unsigned long long mk[RANK_PER]; uint32_t mid[RANK_PER], rank[RANK_PER];
#pragma unroll
        for (int u = 0; u < RANK_PER; ++u) {
            const uint32_t i = min(i0 + u, n - 1u);
            mk[u] = ord_key(raw[i].key); mid[u] = raw[i].id; rank[u] = 0;
        }
        for (uint32_t t0 = 0; t0 < n; t0 += RANK_TILE) {
            const uint32_t m = min((uint32_t)RANK_TILE, n - t0);
            __syncthreads();
            for (uint32_t j = tid; j < m; j += 256) { s_key[j] = ord_key(raw[t0 + j].key); s_id[j] = raw[t0 + j].id; }
            __syncthreads();
            for (uint32_t j = lane; j < m; j += 64) {
                const unsigned long long k = s_key[j]; const uint32_t id = s_id[j];
#pragma unroll
                for (int u = 0; u < RANK_PER; ++u) rank[u] += (k > mk[u] || (k == mk[u] && id < mid[u])) ? 1u : 0u;
            }
        }
#pragma unroll
        for (int u = 0; u < RANK_PER; ++u) {
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) rank[u] += __shfl_xor(rank[u], o);
            if (lane == u && i0 + u < n) { sorted[rank[u]] = raw[i0 + u]; rank_of_id[mid[u]] = rank[u]; }
        }
    }
}

// First fit (Alg. 1 main loop) with the reading of InnerFree given in the header.
// Free rectangle j: fxy[j] = x | y<<16, fwh[j] = w | h<<16, fbin[j].
// box_pos[i] = {bin | turned<<16, bx | by<<16}.
// rotate: a rectangle that cannot take the box upright may take it turned (RotatePacking).
// The loop over the boxes is serial by definition, and it runs in ONE wave, which issues an instruction
// every 4-6 cycles: its cost is the number of instructions of one step.  So
//   - the free list lives in registers, entry j in lane j % 64 of chunk j / 64, up to FREE_CHUNKS * 64 - 2 entries
//     (159 at most for 128 frames of 480 x 272); only the chunks in use are looked at;
//   - a rectangle's sides carry a guard bit each, so that one subtraction tests both (and is the remainder);
//   - the lanes only test their entries: the chosen one is read from its lane, what is left of it is worked out on
//     the scalar unit, with a branch for each outcome, and written back to its lane (v_writelane);
//   - an entry of which nothing is left stays as one without area, which nothing fits; the list is packed anew when it has
//     reached the last lane.  Entries move (a whole-wave DPP shift) only where a used one leaves two in front of others;
//   - a box that fills a bin (three in four of large batches) takes no step.
// Measured, before (every box a step of 170 instructions on the vector unit, entries moved after most of them) / now: the launch of the first fit
// of 745 boxes of 128 frames of 480 x 272 243 / 161 us, the one-launch plan of 139 boxes of 8 frames of 640 x 368 71 / 50 us, of 551
// isolated macroblocks 249-415 / 218-372 us (the one-launch plans with the ranks by waves, below).
// A list that outgrows the registers is written to LDS and stays there: the 64 lanes then test 64
// rectangles at a time; the hardware executes the LDS traffic of a single wave in program order, and
// wave_sync() after every step in which lanes write what other lanes read next keeps the compiler
// from moving LDS accesses across it.
#define FREE_CHUNKS 4
#define FREE_GUARD 0x80008000u           // bin sides are at most 4096
// One wave.  sizes: box i's (wmb | hmb << 16) comes from size_of(i).  Returns through n_bins / overflow.
__device__ __forceinline__ uint32_t lane_from_below(uint32_t v)      // lane l gets lane l-1's value, lane 0 keeps its own
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
}
__device__ __forceinline__ uint32_t lane_from_above(uint32_t v)      // lane l gets lane l+1's value, lane 63 keeps its own
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF, false);
}

// v_writelane_b32: `old` with lane l's value replaced.  The compiler has no builtin for it, so this names its intrinsic, as it is mangled for
// i32; one that mangles it otherwise would report the name as undefined at the library's link, and `lane == l ? value : old` takes its
// place (two instructions more a write).
__device__ int write_lane(int value, int l, int old) __asm("llvm.amdgcn.writelane.i32");

template <bool ROTATE, typename SizeOf>
__device__ __forceinline__ void place_boxes(uint32_t n, SizeOf size_of, uint32_t* fxy, uint32_t* fwh, uint32_t* fbin,
                                            int halo, int S, int max_bins, int free_cap,
                                            uint32_t* __restrict__ box_pos, int& n_bins_out, bool& overflow_out)
{
    const int lane = threadIdx.x & 63;
    const int minside = RH_MB + 2 * halo;
    constexpr int rotate = ROTATE;
    constexpr int REG_MAX = FREE_CHUNKS * 64 - 2;            // a step adds at most 2 entries
    int nfree = 0, nbins = 0;
    uint32_t i = 0, pos0 = 0, pos1 = 0;                      // lane l keeps the position of box (i & ~63) + l
    // rwh: with the guard bits; lanes past the list: no area.  Chunks by name, and no lambda that refers to them:
    // the compiler puts arrays and captured variables into scratch memory here (0.5-0.7 us per box)
    uint32_t rxy0 = 0, rxy1 = 0, rxy2 = 0, rxy3 = 0, rbn0 = 0, rbn1 = 0, rbn2 = 0, rbn3 = 0;
    uint32_t rwh0 = FREE_GUARD, rwh1 = FREE_GUARD, rwh2 = FREE_GUARD, rwh3 = FREE_GUARD;
    bool overflow = false;
    // Results leave in groups of 64: a global store per box would be waited for by the next box's
    // loads (stores and loads share the wave's memory counter), half a microsecond each.
    auto flush = [&](uint32_t upto) {                        // boxes [upto & ~63 ... upto) when upto is not a multiple of 64, else the last 64
        const uint32_t g0 = (upto - 1u) & ~63u;
        if (upto && g0 + lane < upto) { box_pos[2 * (g0 + lane)] = pos0; box_pos[2 * (g0 + lane) + 1] = pos1; }
    };
    // the next 64 box sizes, one per lane, requested 64 boxes ahead
    uint32_t szv = 0, szn = (uint32_t)lane < n ? size_of(lane) : 0u;
    uint32_t ndv = 0;                                        // bw | bh << 16 of these boxes, FREE_GUARD's lower bit: fills a bin of its own
    auto next_sizes = [&]() __attribute__((always_inline)) {
        flush(i);
        szv = szn;
        szn = i + 64 + lane < n ? size_of(i + 64 + lane) : 0u;
        ndv = szv * RH_MB + 2u * halo * 0x10001u;
        const int w = S - (int)(ndv & 0xFFFF), h = S - (int)(ndv >> 16);
        ndv |= max(w, h) < minside ? 0x8000u : 0u;
    };
    auto lane_of = [](uint32_t v, int l) __attribute__((always_inline)) { return (uint32_t)__builtin_amdgcn_readlane((int)v, l); };
    auto with_lane = [](uint32_t v, int l, uint32_t x) __attribute__((always_inline)) { return (uint32_t)write_lane((int)x, l, (int)v); };
    // A box that fills a bin fits no rectangle that another box has left (one side of such a rectangle is at most
    // S - minside), so it opens a bin and leaves nothing.  Such boxes take no step: only the other ones of a group of
    // 64 do (`todo`), and where all of them are placed, the group's full bins are
    // numbered at once.  Where bins or registers might run out within the group, every box takes its step.
    unsigned long long todo = 0, alone = 0, opened = 0;      // alone: the group's boxes that take none; opened: those of the others that opened a bin
    uint32_t g0 = 0;                                         // the group's first box
    int nb0 = 0;                                             // bins before the group; nbins: those and what `opened` says
    int dead = 0;                                            // entries without area among the nfree
    bool grouped = false, more = true;
    auto end_group = [&]() __attribute__((always_inline)) {
        const unsigned long long bins = alone | opened;
        const int b = nb0 + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bins >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bins, 0u));
        const bool mine = alone >> lane & 1ull;
        pos0 = mine ? (uint32_t)b : pos0; pos1 = mine ? 0u : pos1;
        nbins += __builtin_popcountll(alone);
        i = min(g0 + 64u, n);
    };
    auto next_group = [&]() __attribute__((always_inline)) -> bool {
        if (grouped) end_group();
        if (i >= n) return false;
        grouped = true;
        g0 = i;
        next_sizes();
        const unsigned long long all = n - i >= 64u ? ~0ull : (1ull << (n - i)) - 1ull;
        alone = __builtin_amdgcn_ballot_w64((ndv & 0x8000u) != 0) & all;
        if (nbins + __builtin_popcountll(all) > max_bins || nfree + 2 * __builtin_popcountll(all & ~alone) > REG_MAX) alone = 0;
        todo = all & ~alone; opened = 0; nb0 = nbins;
        return true;
    };
    // What is left of a rectangle (ewh, with guard bits, at exy) below and beside a box (need) in its corner: the larger of (right
    // strip, full height) and (bottom strip, full width), plus what is left of the other.  first, last: the survivors in
    // the list's order (the smaller one first), as many as `ni` says.  Conditions are integers: the compiler keeps uniform
    // truth values in vector registers and branches around them.
    uint32_t first_xy, first_wh, last_xy, last_wh, ni;
    auto less = [](uint32_t a, uint32_t b) __attribute__((always_inline)) { return (a - b) >> 31; };       // both below 2^31
    auto rest = [&](uint32_t exy, uint32_t ewh, uint32_t need) __attribute__((always_inline)) {
        const uint32_t rem = ewh - need, rw = rem & 0x7FFF, bhei = rem >> 16 & 0x7FFF;
        const uint32_t fw = ewh & 0x7FFF, fh = ewh >> 16 & 0x7FFF, bw = need & 0xFFFF, bh = need >> 16;
        const bool right_full = rw * fh >= fw * bhei;
        const uint32_t rh = right_full ? fh : bh, bwid = right_full ? bw : fw;
        const uint32_t no_r = less(min(rw, rh), (uint32_t)minside), no_b = less(min(bwid, bhei), (uint32_t)minside);
        const uint32_t b_first = (1u - no_b) & (no_r | less(bwid * bhei, rw * rh));
        const uint32_t Rxy = exy + bw, Rwh = (rw | rh << 16) | FREE_GUARD, Bxy = exy + (need & 0xFFFF0000u), Bwh = (bwid | bhei << 16) | FREE_GUARD;
        first_xy = b_first ? Bxy : Rxy; first_wh = b_first ? Bwh : Rwh; last_xy = b_first ? Rxy : Bxy; last_wh = b_first ? Rwh : Bwh;
        ni = 2u - no_r - no_b;
    };
    // Steps of a list of one chunk.  The entry behind the list's last is the next bin's whole area, so a new bin is an
    // ordinary first fit.  The list's capacity needs no look: its rectangles are
    // disjoint with sides of at least minside, of which a bin holds at most the (S / minside)^2 that free_cap counts.
    const uint32_t whole = FREE_GUARD | (uint32_t)S | (uint32_t)S << 16;
    // The list to LDS without the entries without area, in any case less than free_cap, and back
#define PACK(c) {                                                                                   \
        const bool has = 64 * c + lane < nfree && rwh##c != FREE_GUARD;                             \
        const unsigned long long live = __builtin_amdgcn_ballot_w64(has);                           \
        const int j = packed + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(live >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)live, 0u));    \
        if (has) { fxy[j] = rxy##c; fwh[j] = rwh##c & ~FREE_GUARD; fbin[j] = rbn##c; }              \
        packed += __builtin_popcountll(live); }
#define PACKED() { wave_sync(); nfree = packed; packed = 0; dead = 0; }
#define TAKE(c) {                                                                                   \
        const int j = 64 * c + lane;                                                                \
        rwh##c = FREE_GUARD;                                                                        \
        if (j < nfree) { rxy##c = fxy[j]; rwh##c = fwh[j] | FREE_GUARD; rbn##c = fbin[j]; } }
    int packed = 0;
    do {
        for (;;) {
            if (todo == 0) {
                more = next_group();
                if (!more) break;
            }
            if (nfree >= 61 && dead >= 16) { PACK(0) PACKED() TAKE(0) wave_sync(); }      // the last lanes are in use
            // as many steps as lanes and bins are there for in any case
            int steps = min(min(__builtin_popcountll(todo), (62 - nfree) / 2), max_bins - nbins - __builtin_popcountll(alone));
            if (steps <= 0 && todo != 0) break;
            // what a step needs of its box is at hand before the step: its number in the group, its sides, the bin it would open
            int k = 0;
            uint32_t need = 0;
#define NEXT_BOX() {                                                                                \
                k = __builtin_ctzll(todo | 1ull << 63);                                             \
                need = lane_of(ndv, k) & ~0x8000u;                                                  \
                const int bin = nbins + __builtin_popcountll(alone & ((1ull << k) - 1ull));         \
                rxy0 = with_lane(rxy0, nfree, 0u); rwh0 = with_lane(rwh0, nfree, whole); rbn0 = with_lane(rbn0, nfree, (uint32_t)bin); }
            NEXT_BOX()
            for (; steps > 0; --steps) {
                bool fit = ((rwh0 - need) & FREE_GUARD) == FREE_GUARD;
                const uint32_t needt = need >> 16 | need << 16;
                if constexpr (ROTATE) fit = fit | (((rwh0 - needt) & FREE_GUARD) == FREE_GUARD);
                const int at = __builtin_ctzll(__builtin_amdgcn_ballot_w64(fit));
                const uint32_t exy = lane_of(rxy0, at), ewh = lane_of(rwh0, at), eb = lane_of(rbn0, at);
                uint32_t turned = 0;
                if constexpr (ROTATE) {                          // upright whenever that fits
                    const bool up = ((ewh - need) & FREE_GUARD) == FREE_GUARD;
                    need = up ? need : needt; turned = up ? 0u : 0x10000u;
                }
                pos0 = with_lane(pos0, k, eb | turned); pos1 = with_lane(pos1, k, exy);
                rest(exy, ewh, need);
                const uint32_t old = min((uint32_t)(nfree - at), 1u), fresh = 1u - old;      // fresh: what is left of a new bin goes to the list's end
                nbins += (int)fresh; opened |= (unsigned long long)fresh << k;
                if (ni == 2u) {
                    if (old) {                                   // the entries behind `at` move up by one
                        const uint32_t dxy = lane_from_below(rxy0), dwh = lane_from_below(rwh0), dbn = lane_from_below(rbn0);
                        const bool up = lane > at;
                        rxy0 = up ? dxy : rxy0; rwh0 = up ? dwh : rwh0; rbn0 = up ? dbn : rbn0;
                    }
                    rxy0 = with_lane(rxy0, at + 1, last_xy); rwh0 = with_lane(rwh0, at + 1, last_wh); rbn0 = with_lane(rbn0, at + 1, eb);
                }
                rxy0 = with_lane(rxy0, at, first_xy); rwh0 = with_lane(rwh0, at, ni ? first_wh : FREE_GUARD);
                dead += (int)(old & less(ni, 1u));
                nfree += (int)(ni - min(ni, old));
                todo &= todo - 1;
                NEXT_BOX()
            }
#undef NEXT_BOX
        }
        if (lane >= nfree) rwh0 = FREE_GUARD;                    // without the new bin's entry
        // ---- several chunks ----
        while (more && !overflow) {
            if (nfree > REG_MAX || (todo == 0 && dead >= 64)) {
                PACK(0) PACK(1) PACK(2) PACK(3) PACKED()
                TAKE(0) TAKE(1) TAKE(2) TAKE(3)
                wave_sync();
                if (nfree > REG_MAX - 8 || nfree < 40) break;
            }
            if (todo == 0) { more = next_group(); continue; }
            const int k = __builtin_ctzll(todo);
            todo &= todo - 1;
            uint32_t need = lane_of(ndv, k) & ~0x8000u;
            const uint32_t needt = need >> 16 | need << 16;
#define FITS(c)                                                                                     \
            bool fit##c = ((rwh##c - need) & FREE_GUARD) == FREE_GUARD;                                 \
            if constexpr (ROTATE) fit##c = fit##c | (((rwh##c - needt) & FREE_GUARD) == FREE_GUARD);
            FITS(0) FITS(1) FITS(2) FITS(3)
#undef FITS
#define PUT1(c, j, xy, wh) if (((j) >> 6) == c) { rxy##c = with_lane(rxy##c, (j) & 63, xy); rwh##c = with_lane(rwh##c, (j) & 63, wh); rbn##c = with_lane(rbn##c, (j) & 63, eb); }
#define PUT(j, xy, wh) do { PUT1(0, j, xy, wh) else PUT1(1, j, xy, wh) else PUT1(2, j, xy, wh) else PUT1(3, j, xy, wh) } while (0)
            if (__builtin_amdgcn_ballot_w64(fit0 | fit1 | fit2 | fit3) == 0) {      // a new bin: what is left of it goes to the list's end
                const uint32_t eb = (uint32_t)nbins + (uint32_t)__builtin_popcountll(alone & ((1ull << k) - 1ull));
                if ((int)eb >= max_bins) { overflow = true; i = g0 + k; break; }
                ++nbins; opened |= 1ull << k;
                pos0 = with_lane(pos0, k, eb); pos1 = with_lane(pos1, k, 0u);
                rest(0u, whole, need);
                if (ni >= 1u) { PUT(nfree, first_xy, first_wh); ++nfree; }
                if (ni == 2u) { PUT(nfree, last_xy, last_wh); ++nfree; }
                continue;
            }
            int at = -1;
            uint32_t exy = 0, ewh = 0, eb = 0;
#define FIRST(c)                                                                                    \
            if (at < 0) {                                                                               \
                const unsigned long long m = __builtin_amdgcn_ballot_w64(fit##c);                       \
                if (m) {                                                                                \
                    const int l = __builtin_ctzll(m);                                                   \
                    at = 64 * c + l;                                                                    \
                    exy = lane_of(rxy##c, l); ewh = lane_of(rwh##c, l); eb = lane_of(rbn##c, l);        \
                }                                                                                       \
            }
            FIRST(0) FIRST(1) FIRST(2) FIRST(3)
#undef FIRST
            uint32_t turned = 0;
            if constexpr (ROTATE) if (((ewh - need) & FREE_GUARD) != FREE_GUARD) { need = needt; turned = 0x10000u; }      // upright whenever that fits
            pos0 = with_lane(pos0, k, eb | turned); pos1 = with_lane(pos1, k, exy);
            rest(exy, ewh, need);
            if (ni == 0) { ++dead; first_wh = FREE_GUARD; }      // an entry without area
            if (ni == 2) {
#define UP(c, below)                                                                                \
                if (64 * c <= nfree && c >= (at >> 6)) {                                                \
                    uint32_t xy = lane_from_below(rxy##c), wh = lane_from_below(rwh##c), bn = lane_from_below(rbn##c);     \
                    if (c > (at >> 6)) {                                                                \
                        xy = with_lane(xy, 0, lane_of(rxy##below, 63)); wh = with_lane(wh, 0, lane_of(rwh##below, 63));    \
                        bn = with_lane(bn, 0, lane_of(rbn##below, 63));                                 \
                    }                                                                                   \
                    const bool mv = lane + 64 * c > at;                                                 \
                    rxy##c = mv ? xy : rxy##c; rwh##c = mv ? wh : rwh##c; rbn##c = mv ? bn : rbn##c;    \
                }
                UP(3, 2) UP(2, 1) UP(1, 0) UP(0, 0)              // the entries behind `at` move up by one
#undef UP
                PUT(at + 1, last_xy, last_wh);
                ++nfree;
            }
            PUT(at, first_xy, first_wh);
#undef PUT
#undef PUT1
        }
    } while (more && !overflow && nfree < 40);
    // ---- the list has outgrown the registers: it moves to LDS for the rest of the boxes ----
    if (more && !overflow) {                                 // not amid a group that leaves out boxes
        if (todo == 0) end_group();
        else i = g0 + (uint32_t)__builtin_ctzll(todo);
        PACK(0) PACK(1) PACK(2) PACK(3) PACKED()
    }
#undef PACK
#undef PACKED
#undef TAKE
    for (; i < n && !overflow; ++i) {
        if ((i & 63u) == 0) next_sizes();
        const uint32_t sz = lane_of(szv, (int)(i & 63u));
        int bw = RH_MB * (int)(sz & 0xFFFF) + 2 * halo, bh = RH_MB * (int)(sz >> 16) + 2 * halo;
        // first rectangle, in list order, that fits: every lane reads one entry whole, the winner's
        // fields are then taken from its lane
        uint32_t at = NONE, exy = 0, ewh = 0, ebin = 0;
        for (int base = 0; base < nfree; base += 64) {
            const int j = base + lane;
            uint32_t wh = 0, xy = 0, bn = 0;
            if (j < nfree) { wh = fwh[j]; xy = fxy[j]; bn = fbin[j]; }
            const int w = (int)(wh & 0xFFFF), h = (int)(wh >> 16);
            const bool fit = j < nfree && ((w >= bw && h >= bh) || (rotate && w >= bh && h >= bw));
            const unsigned long long m = __ballot(fit);
            if (m) {
                const int l = __ffsll((long long)m) - 1;
                at = (uint32_t)(base + l);
                exy = (uint32_t)__builtin_amdgcn_readlane((int)xy, l); ewh = (uint32_t)__builtin_amdgcn_readlane((int)wh, l);
                ebin = (uint32_t)__builtin_amdgcn_readlane((int)bn, l);
                break;
            }
        }
        int fx, fy, fw, fh, fb, cur_n;
        if (at == NONE) {
            if (nbins >= max_bins || nfree + 2 > free_cap) { overflow = true; break; }
            at = nfree; fx = 0; fy = 0; fw = S; fh = S; fb = nbins++; cur_n = nfree + 1;
        } else {
            fx = exy & 0xFFFF; fy = exy >> 16; fw = ewh & 0xFFFF; fh = ewh >> 16; fb = ebin;
            cur_n = nfree;
            if (nfree + 1 > free_cap) { overflow = true; break; }
        }
        const bool turned = !(fw >= bw && fh >= bh);         // upright whenever that fits
        if (turned) { const int t = bw; bw = bh; bh = t; }   // occupied size
        if (lane == (int)(i & 63u)) { pos0 = (uint32_t)fb | (turned ? 0x10000u : 0u); pos1 = (uint32_t)fx | ((uint32_t)fy << 16); }
        const int ar = (fw - bw) * fh, ab = fw * (fh - bh);
        int rx = fx + bw, ry = fy, rw = fw - bw, rh, bx = fx, by = fy + bh, bwid, bhei = fh - bh;
        if (ar >= ab) { rh = fh; bwid = bw; } else { rh = bh; bwid = fw; }
        const bool keep_r = rw >= minside && rh >= minside, keep_b = bwid >= minside && bhei >= minside;
        uint32_t ixy[2] = {0, 0}, iwh[2] = {0, 0}; int ni = 0;
        const uint32_t Rxy = rx | (ry << 16), Rwh = rw | (rh << 16), Bxy = bx | (by << 16), Bwh = bwid | (bhei << 16);
        if (keep_r && keep_b) {
            if (bwid * bhei < rw * rh) { ixy[0] = Bxy; iwh[0] = Bwh; ixy[1] = Rxy; iwh[1] = Rwh; }
            else                       { ixy[0] = Rxy; iwh[0] = Rwh; ixy[1] = Bxy; iwh[1] = Bwh; }
            ni = 2;
        } else if (keep_r) { ixy[0] = Rxy; iwh[0] = Rwh; ni = 1; }
        else if (keep_b)   { ixy[0] = Bxy; iwh[0] = Bwh; ni = 1; }
        // the survivors replace entry `at` in place: shift the tail by ni - 1
        const int delta = ni - 1, first = (int)at + 1;
        if (delta > 0) {
            for (int hi = cur_n; hi > first; hi -= 64) {         // from the top down: a chunk is read whole before it is written
                const int j = hi - 1 - lane;
                uint32_t a = 0, b = 0, c = 0;
                if (j >= first) { a = fxy[j]; b = fwh[j]; c = fbin[j]; }
                wave_sync();
                if (j >= first) { fxy[j + 1] = a; fwh[j + 1] = b; fbin[j + 1] = c; }
                wave_sync();
            }
        } else if (delta < 0) {
            for (int lo = first; lo < cur_n; lo += 64) {
                const int j = lo + lane;
                uint32_t a = 0, b = 0, c = 0;
                if (j < cur_n) { a = fxy[j]; b = fwh[j]; c = fbin[j]; }
                wave_sync();
                if (j < cur_n) { fxy[j - 1] = a; fwh[j - 1] = b; fbin[j - 1] = c; }
                wave_sync();
            }
        }
        if (lane < ni) { fxy[at + lane] = ixy[lane]; fwh[at + lane] = iwh[lane]; fbin[at + lane] = fb; }
        wave_sync();
        nfree = cur_n + delta;
    }
    flush(i);                                                // i = boxes placed
    // boxes that did not fit (only after an overflow)
    for (uint32_t j = i + lane; j < n; j += 64) { box_pos[2 * j] = RH_NO_BIN; box_pos[2 * j + 1] = 0; }
    n_bins_out = nbins; overflow_out = overflow;
}

// pcount: 0 boxes, 1 bins, 2 overflow, 3 boxes appended by the labelling kernel.  Every plan of several launches
// clears the append counter itself: were it left at 0 by the plan before, one lost launch would
// make all later plans append behind stale boxes and past the end of raw.
__global__ void k_plan_zero(uint32_t* pcount) { pcount[3] = 0; }

__global__ __launch_bounds__(64) void k_plan_place(const rh_rawbox* __restrict__ sorted, uint32_t* pcount,
                                                   int halo, int S, int max_bins, int free_cap, int rotate,
                                                   uint32_t* __restrict__ box_pos)
{
    extern __shared__ uint32_t sm[];
    int nbins; bool overflow;
    const uint32_t n = pcount[3];
    auto size_of = [&](uint32_t i) { return (uint32_t)sorted[i].wmb | ((uint32_t)sorted[i].hmb << 16); };
    if (rotate) place_boxes<true>(n, size_of, sm, sm + free_cap, sm + 2 * free_cap, halo, S, max_bins, free_cap, box_pos, nbins, overflow);
    else place_boxes<false>(n, size_of, sm, sm + free_cap, sm + 2 * free_cap, halo, S, max_bins, free_cap, box_pos, nbins, overflow);
    if (threadIdx.x == 0) { pcount[0] = n; pcount[1] = nbins; pcount[2] = overflow ? 1u : 0u; }
}

// Placement rows of box i and of selected macroblock i (Alg. 1's output).
__device__ __forceinline__ void emit_rows(uint32_t i, uint32_t n, uint32_t n_sel, const rh_rawbox* __restrict__ sorted,
                                          const uint32_t* __restrict__ box_pos, const uint32_t* __restrict__ list,
                                          const uint32_t* __restrict__ owner_id, const uint32_t* __restrict__ rank_of_id,
                                          int mbw, int per, int halo, rh_box* __restrict__ boxes, rh_mbplace* __restrict__ places)
{
    if (i < n) {
        const rh_rawbox b = sorted[i];
        rh_box o;
        o.frame = b.frame; o.mbx0 = b.mbx0; o.mby0 = b.mby0; o.wmb = (uint8_t)b.wmb; o.hmb = (uint8_t)b.hmb;
        o.rot = (uint8_t)((box_pos[2 * i] >> 16) & 1u); o.pad0 = 0; o.bin = (uint16_t)(box_pos[2 * i] & 0xFFFFu);
        o.bx = (uint16_t)(box_pos[2 * i + 1] & 0xFFFF); o.by = (uint16_t)(box_pos[2 * i + 1] >> 16);
        o.pad1 = 0; o.id = b.id;
        boxes[i] = o;
    }
    if (i < n_sel) {
        const uint32_t g = list[i], rk = rank_of_id[owner_id[g]];
        const rh_rawbox b = sorted[rk];
        const uint32_t in = g % (uint32_t)per;
        const int y = in / mbw, x = in - y * mbw;
        rh_mbplace p;
        p.mb_id = g; p.box = rk; p.bin = (uint16_t)(box_pos[2 * rk] & 0xFFFFu);
        const bool placed = p.bin != RH_NO_BIN;
        const bool turned = (box_pos[2 * rk] >> 16) & 1u;
        const int dx = halo + RH_MB * (x - b.mbx0), dy = halo + RH_MB * (y - b.mby0);
        p.px = placed ? (uint16_t)((box_pos[2 * rk + 1] & 0xFFFF) + (turned ? dy : dx)) : 0;
        p.py = placed ? (uint16_t)((box_pos[2 * rk + 1] >> 16) + (turned ? dx : dy)) : 0;
        p.rot = turned ? 1 : 0;
        places[i] = p;
    }
}

__global__ __launch_bounds__(256) void k_plan_emit(const rh_rawbox* __restrict__ sorted,
                                                   const uint32_t* __restrict__ box_pos,
                                                   const uint32_t* __restrict__ pcount,
                                                   const uint32_t* __restrict__ list,
                                                   const uint32_t* __restrict__ n_sel_p,
                                                   const uint32_t* __restrict__ owner_id,
                                                   const uint32_t* __restrict__ rank_of_id, int mbw, int per,
                                                   int halo, rh_box* __restrict__ boxes,
                                                   rh_mbplace* __restrict__ places, uint32_t* __restrict__ counts)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    const uint32_t n = pcount[0], n_sel = *n_sel_p;
    if (i == 0) { counts[0] = n; counts[1] = pcount[1]; counts[2] = pcount[2]; counts[3] = n_sel; }
    emit_rows(i, n, n_sel, sorted, box_pos, list, owner_id, rank_of_id, mbw, per, halo, boxes, places);
}

// ------------------------------------------------------------------------------------------------
// The whole plan in ONE launch of one 1024-thread workgroup, for frames of at most 64 x 64
// macroblocks (1024 x 1024 pixels; the paper's streams are 640 x 360).  A plan is a few hundred
// boxes: five dependent launches cost more than the work itself.
//   A  label + bound + partition: one wave per frame (16 frames at a time), no barriers.  Lane y
//      holds row y of the frame's selection as a 64-bit mask.  A region grows from its first
//      macroblock in raster order (= its smallest index, its label): rows exchange masks with the
//      rows above and below, spread by one column (8-connectivity: the union of the three, 4: only
//      the row's own), and fill whole horizontal runs with two carry-propagating additions, until
//      nothing changes.  The region's bounding box is cut on the T x T grid; one lane per cell
//      walks the cell's rows (masks fetched from the row lanes), tightens the bounds, adds the
//      importance values in ascending index (fp32, from an LDS copy of the frame's map) and
//      writes the box and its macroblocks' owner.
//   B  rank by counting over all threads (keys in LDS for up to PF_KEYS boxes)
//   C  first fit by wave 0 (place_boxes)
//   D  placement rows by all threads
#define PF_THREADS 1024
#define PF_WAVES (PF_THREADS / 64)
#define PF_KEYS 2048
// More frames: phases in launches of their own.  Up to 16 the labelling is one round of waves here.  Select + plan + gather in us,
// one launch / several: 480 x 272, 6 frames 36.1 / 44.5, 12: 48.3 / 52.5, 16: 55.1 / 57.5, 17: 57.1 / 57.2, 24: 70.9 / 64.4; 640 x 368,
// 16: 73.5 / 72.5, 17: 74.0 / 72.0; 320 x 192, 17: 40.0 / 41.1.  Where there are many boxes, a number that the host does not know, several
// are faster: scattered macroblocks, 16 frames of 480 x 272 (551 boxes) 232 / 210, of 640 x 368 (957) 408 / 346.
#define PF_FRAMES 16
#define PF_MAX_PER 2304                   // 16 waves x per x 4 B of importance <= 144 KB

typedef unsigned long long u64;

__device__ __forceinline__ u64 fill_runs(u64 n, u64 m)     // extend the bits of n (a subset of m) along the runs of ones of m
{
    const u64 up = ((m + n) ^ m) & m;                        // a carry runs from every seed to the end of its run
    const u64 rm = __brevll(m), rn = __brevll(n);
    const u64 dn = __brevll(((rm + rn) ^ rm) & rm);
    return n | up | dn;
}

// 64-bit values of the lanes beside this one (0 past the ends), of one lane, and the union over all lanes: by DPP
// and lane reads, a few cycles each, where a shuffle goes through LDS (about 100) - a region takes one
// exchange for every row that it spans
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ u64 dpp64(u64 v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xF, false);
    return (u64)hi << 32 | lo;
}
__device__ __forceinline__ u64 row_above(u64 v) { return dpp64<0x138 /* wave_shr:1 */>(v); }
__device__ __forceinline__ u64 row_below(u64 v) { return dpp64<0x130 /* wave_shl:1 */>(v); }
__device__ __forceinline__ u64 row_of(u64 v, int l)
{
    return (u64)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
}
__device__ __forceinline__ u64 rows_or(u64 v)
{
    v |= dpp64<0x111 /* row_shr:1 */>(v); v |= dpp64<0x112>(v); v |= dpp64<0x114>(v); v |= dpp64<0x118>(v);
    v |= dpp64<0x142 /* row_bcast:15 */, 0xA>(v); v |= dpp64<0x143 /* row_bcast:31 */, 0xC>(v);
    return row_of(v, 63);
}

// The sum of all lanes' values
__device__ __forceinline__ uint32_t lane_sum(uint32_t v)
{
#define STEP(ctrl, rows) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xF, false)
    STEP(0x111 /* row_shr:1 */, 0xF); STEP(0x112, 0xF); STEP(0x114, 0xF); STEP(0x118, 0xF);
    STEP(0x142 /* row_bcast:15 */, 0xA); STEP(0x143 /* row_bcast:31 */, 0xC);
#undef STEP
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

struct plan_args {
    const uint8_t* mask; const float* imp; const uint32_t* list; const uint32_t* n_sel;
    int F, mbw, mbh, conn, T, sort_policy, halo, S, max_bins, free_cap, rotate;
    uint32_t* owner_id; uint32_t* rank_of_id; rh_rawbox* raw; rh_rawbox* sorted; uint32_t* box_pos;
    rh_box* boxes; rh_mbplace* places; uint32_t* counts;
};

// Phase A for frame f, one wave: its regions, bounds and boxes.  append(k): first of k new slots of a.raw.
template <typename Append>
__device__ __forceinline__ void frame_boxes(const plan_args& a, int f, float* simp, Append append)
{
    const int lane = threadIdx.x & 63, mbw = a.mbw, mbh = a.mbh, per = mbw * mbh, T = a.T;
    const size_t base = (size_t)f * per;
    for (int i = lane; i < per; i += 64) simp[i] = a.imp[base + i];
    u64 m = 0;
    for (int y = 0; y < mbh; y += 8) {                   // eight rows' loads in flight at a time
        uint8_t v8[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v8[u] = (lane < mbw && y + u < mbh) ? a.mask[base + (size_t)(y + u) * mbw + lane] : (uint8_t)0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const u64 row = __ballot(v8[u] != 0);
            if (lane == y + u) m = row;
        }
    }
    wave_sync();                                         // simp is read by other lanes below
    // Macroblocks without a neighbour are regions and boxes of one macroblock: every row writes its own at
    // the same time.  (One region after the other took 2 us each, half of them with scattered importance.)
    u64 iso;
    {
        const u64 up = row_above(m), dn = row_below(m);
        const u64 col = a.conn == 8 ? m | up | dn : m;
        iso = m & ~((col << 1) | (col >> 1) | up | dn);
    }
    u64 rem = m & ~iso;
    for (;;) {
        const bool has = iso != 0;
        const u64 hm = __ballot(has);
        if (!hm) break;
        uint32_t slot0 = 0;
        if (lane == 0) slot0 = append((uint32_t)__popcll(hm));
        slot0 = __shfl(slot0, 0);
        if (has) {
            const int x = __ffsll((long long)iso) - 1, g = lane * mbw + x;
            iso &= iso - 1;
            rh_rawbox b;
            b.frame = f; b.mbx0 = x; b.mby0 = lane; b.wmb = 1; b.hmb = 1;
            b.id = (uint32_t)(base + g); b.sum = __fadd_rn(0.0f, simp[g]);
            b.key = a.sort_policy == RH_SORT_AREA ? 1.0 : (double)b.sum;
            a.raw[slot0 + (uint32_t)__popcll(hm & ((1ull << lane) - 1ull))] = b;
            a.owner_id[base + g] = b.id;
        }
    }
    for (;;) {
        const u64 rows_left = __ballot(rem != 0);
        if (!rows_left) break;
        const int ys = __ffsll((long long)rows_left) - 1;
        const u64 seed_row = row_of(rem, ys);
        u64 comp = lane == ys ? (seed_row & (~seed_row + 1)) : 0;           // lowest set bit: the region's label
        for (;;) {                                       // RegionProps: grow until stable
            const u64 up = row_above(comp), dn = row_below(comp);
            u64 n;
            if (a.conn == 8) { n = comp | up | dn; n |= (n << 1) | (n >> 1); }
            else n = comp | up | dn | (comp << 1) | (comp >> 1);
            n = fill_runs((n & m) | comp, m);
            const bool changed = n != comp;
            comp = n;
            if (!__any(changed)) break;
        }
        rem &= ~comp;
        // Bound
        const u64 rows_in = __ballot(comp != 0);
        const int y0 = __ffsll((long long)rows_in) - 1, y1 = 63 - __clzll((long long)rows_in);
        const u64 cols = rows_or(comp);
        const int x0 = __ffsll((long long)cols) - 1, x1 = 63 - __clzll((long long)cols);
        // Partition: cells of the T x T grid anchored at (x0, y0), one lane per cell
        const int ncx = (x1 - x0) / T + 1, ncy = (y1 - y0) / T + 1, cells = ncx * ncy;
        for (int c0 = 0; c0 < cells; c0 += 64) {         // uniform over the wave
            const int c = c0 + lane;
            const bool active = c < cells;
            const int cy = active ? c / ncx : 0, cx = active ? c - cy * ncx : 0;
            const int ra = y0 + cy * T, rb = min(ra + T - 1, y1), ca = x0 + cx * T, cb = min(ca + T - 1, x1);
            const u64 cmask = ((cb - ca + 1) >= 64 ? ~0ull : ((1ull << (cb - ca + 1)) - 1ull)) << ca;
            int leader = -1, bx0 = 64, bx1 = -1, by0 = 64, by1 = -1;
            float sum = 0.0f;
            const int span = min(T, y1 - y0 + 1);       // rows a cell can have: uniform
            for (int rr = 0; rr < span; ++rr) {
                const int r = ra + rr;
                const u64 rowbits = __shfl(comp, (active && r <= rb) ? r : 0);     // every lane takes part
                u64 bits = (active && r <= rb) ? (rowbits & cmask) : 0;
                if (bits) {
                    if (leader < 0) { leader = r * mbw + (__ffsll((long long)bits) - 1); by0 = r; }
                    by1 = r;
                    bx0 = min(bx0, __ffsll((long long)bits) - 1); bx1 = max(bx1, 63 - __clzll((long long)bits));
                    while (bits) {                       // ascending column = ascending flat index
                        const int x = __ffsll((long long)bits) - 1;
                        bits &= bits - 1;
                        sum = __fadd_rn(sum, simp[r * mbw + x]);
                        a.owner_id[base + r * mbw + x] = (uint32_t)(base + leader);
                    }
                }
            }
            const bool has = leader >= 0;
            const u64 hm = __ballot(has);
            uint32_t slot0 = 0;
            if (lane == 0 && hm) slot0 = append((uint32_t)__popcll(hm));
            slot0 = __shfl(slot0, 0);
            if (has) {
                rh_rawbox b;
                b.frame = f; b.mbx0 = bx0; b.mby0 = by0; b.wmb = bx1 - bx0 + 1; b.hmb = by1 - by0 + 1;
                b.id = (uint32_t)(base + leader); b.sum = sum;
                const int area = (bx1 - bx0 + 1) * (by1 - by0 + 1);
                b.key = a.sort_policy == RH_SORT_AREA ? (double)area : (double)sum / (double)area;
                a.raw[slot0 + (uint32_t)__popcll(hm & ((1ull << lane) - 1ull))] = b;
            }
        }
    }
}

// Phase A in a launch of its own, one frame per workgroup of one wave
__global__ __launch_bounds__(64) void k_plan_regions(plan_args a, uint32_t* pcount)
{
    extern __shared__ float simp[];
    frame_boxes(a, blockIdx.x, simp, [&](uint32_t k) { return atomicAdd(&pcount[3], k); });
}

__global__ __launch_bounds__(PF_THREADS) void k_plan_fused(plan_args a)
{
    extern __shared__ __attribute__((aligned(16))) uint32_t dyn[];
    __shared__ uint32_t s_nraw, s_nbins, s_overflow;
    __shared__ uint32_t s_sz[PF_KEYS];                       // sizes of the sorted boxes, for the first fit
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int mbw = a.mbw, per = mbw * a.mbh;
    if (tid == 0) s_nraw = 0;
    __syncthreads();

    // ---------------- A: regions and boxes, one wave per frame ----------------
    float* simp = (float*)dyn + (size_t)wave * per;
    for (int f = wave; f < a.F; f += PF_WAVES) {
        frame_boxes(a, f, simp, [&](uint32_t k) { return atomicAdd(&s_nraw, k); });
        wave_sync();                                         // before the next frame overwrites simp
    }
    __threadfence_block();
    __syncthreads();
    const uint32_t n = s_nraw, n_sel = *a.n_sel;

    // ---------------- B: rank by counting ----------------
    u64* s_key = (u64*)dyn;
    uint32_t* s_id = (uint32_t*)(s_key + PF_KEYS);
    const bool keys_in_lds = n <= PF_KEYS;
    if (keys_in_lds)
        for (uint32_t j = tid; j < n; j += PF_THREADS) { s_key[j] = ord_key(a.raw[j].key); s_id[j] = a.raw[j].id; }
    __syncthreads();
    if (keys_in_lds) {
        // a wave ranks two boxes at a time, its lanes compare them with 64 others each step (a thread per box, eight keys at a
        // time: 27 us of 551 boxes, 7.5 of 139; their plans 314 -> 301 and 53 -> 49 us)
        for (uint32_t i0 = wave * 2; i0 < n; i0 += PF_WAVES * 2) {
            const uint32_t i1 = min(i0 + 1, n - 1u), d0 = s_id[i0], d1 = s_id[i1];
            const u64 k0 = s_key[i0], k1 = s_key[i1];
            uint32_t r0 = 0, r1 = 0;
            for (uint32_t j = lane; j < n; j += 64) {
                const u64 k = s_key[j]; const uint32_t id = s_id[j];
                r0 += (k > k0 || (k == k0 && id < d0)) ? 1u : 0u;
                r1 += (k > k1 || (k == k1 && id < d1)) ? 1u : 0u;
            }
            r0 = lane_sum(r0 | r1 << 16);                    // at most PF_KEYS each
            const uint32_t rank = lane ? r0 >> 16 : r0 & 0xFFFFu;
            const rh_rawbox* me = a.raw + min(i0 + lane, n - 1u);
            if (i0 + lane < n && lane < 2) {
                a.sorted[rank] = *me; a.rank_of_id[me->id] = rank;
                s_sz[rank] = (uint32_t)me->wmb | ((uint32_t)me->hmb << 16);
            }
        }
    } else {
        for (uint32_t i = tid; i < n; i += PF_THREADS) {
            const rh_rawbox me = a.raw[i];
            uint32_t rank = 0;
            for (uint32_t j = 0; j < n; ++j) rank += box_before(a.raw[j].key, a.raw[j].id, me.key, me.id) ? 1u : 0u;
            a.sorted[rank] = me; a.rank_of_id[me.id] = rank;
            if (rank < PF_KEYS) s_sz[rank] = (uint32_t)me.wmb | ((uint32_t)me.hmb << 16);
        }
    }
    __threadfence_block();
    __syncthreads();                                         // keys are dead: the free list takes their place

    // ---------------- C: first fit, wave 0 ----------------
    if (wave == 0) {
        int nbins; bool overflow;
        auto size_of = [&](uint32_t i) { return i < PF_KEYS ? s_sz[i] : ((uint32_t)a.sorted[i].wmb | ((uint32_t)a.sorted[i].hmb << 16)); };
        uint32_t* fl = dyn;
        if (a.rotate) place_boxes<true>(n, size_of, fl, fl + a.free_cap, fl + 2 * a.free_cap, a.halo, a.S, a.max_bins, a.free_cap, a.box_pos, nbins, overflow);
        else place_boxes<false>(n, size_of, fl, fl + a.free_cap, fl + 2 * a.free_cap, a.halo, a.S, a.max_bins, a.free_cap, a.box_pos, nbins, overflow);
        if (lane == 0) { s_nbins = (uint32_t)nbins; s_overflow = overflow ? 1u : 0u; }
    }
    __threadfence_block();
    __syncthreads();

    // ---------------- D: placement rows ----------------
    if (tid == 0) { a.counts[0] = n; a.counts[1] = s_nbins; a.counts[2] = s_overflow; a.counts[3] = n_sel; }
    const uint32_t top = n > n_sel ? n : n_sel;
    for (uint32_t i = tid; i < top; i += PF_THREADS)
        emit_rows(i, n, n_sel, a.sorted, a.box_pos, a.list, a.owner_id, a.rank_of_id, mbw, per, a.halo, a.boxes, a.places);
}

rh_status rh_plan_init(rh_ctx* ctx)
{
    // The planning kernels may need more dynamic LDS than the default limit.  The attribute belongs
    // to the kernel, not to the context: it is raised to what the largest admissible context needs
    // (rh_create bounds the sizes below 150 KB), so contexts of different sizes can coexist.
    RH_HIP(ctx, hipFuncSetAttribute((const void*)k_plan_label, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024));
    RH_HIP(ctx, hipFuncSetAttribute((const void*)k_plan_place, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024));
    RH_HIP(ctx, hipFuncSetAttribute((const void*)k_plan_fused, hipFuncAttributeMaxDynamicSharedMemorySize, 144 * 1024));
    return RH_OK;
}

rh_status rh_launch_plan(rh_ctx* ctx, int F, const float* imp, const uint8_t* mask,
                         const uint32_t* list, const uint32_t* n_sel,
                         rh_box* boxes, rh_mbplace* places, uint32_t* counts)
{
    const int per = ctx->per, total = per * F;
    uint32_t* box_pos = ctx->pcount + 8;
    plan_args a;
    a.mask = mask; a.imp = imp; a.list = list; a.n_sel = n_sel;
    a.F = F; a.mbw = ctx->mbw; a.mbh = ctx->mbh; a.conn = ctx->cfg.connectivity; a.T = ctx->T;
    a.sort_policy = ctx->cfg.sort_policy; a.halo = ctx->cfg.halo; a.S = ctx->cfg.bin_size; a.max_bins = ctx->cfg.max_bins;
    a.free_cap = ctx->free_cap; a.rotate = ctx->cfg.rotate;
    a.owner_id = ctx->owner_id; a.rank_of_id = ctx->rank_of_id; a.raw = ctx->raw; a.sorted = ctx->sorted; a.box_pos = box_pos;
    a.boxes = boxes; a.places = places; a.counts = counts;
    const bool rows64 = ctx->mbw <= 64 && ctx->mbh <= 64 && per <= PF_MAX_PER;
    if (rows64 && F <= PF_FRAMES) {
        // the usual batch: everything in one launch
        size_t lds = (size_t)PF_WAVES * per * 4;
        if (lds < (size_t)PF_KEYS * 12) lds = (size_t)PF_KEYS * 12;
        if (lds < (size_t)ctx->free_cap * 12) lds = (size_t)ctx->free_cap * 12;
        rh_prof_scope ps(ctx, RH_PROF_PLAN, 1);
        hipLaunchKernelGGL(k_plan_fused, dim3(1), dim3(PF_THREADS), lds, ctx->stream, a);
        RH_HIP(ctx, hipGetLastError());
        return RH_OK;
    }
    // A launch that fails ends the call: the kernels behind it would read what it has not written.
#define LAUNCHED() RH_HIP(ctx, hipGetLastError())
    rh_prof_scope ps(ctx, RH_PROF_PLAN, 5);
    hipLaunchKernelGGL(k_plan_zero, dim3(1), dim3(1), 0, ctx->stream, ctx->pcount);
    LAUNCHED();
    if (rows64) {
        hipLaunchKernelGGL(k_plan_regions, dim3(F), dim3(64), (size_t)per * 4, ctx->stream, a, ctx->pcount);
    } else {
        const int imp_in_lds = (size_t)per * 20 <= 150 * 1024;
        hipLaunchKernelGGL(k_plan_label, dim3(F), dim3(256), (size_t)per * (imp_in_lds ? 20 : 16), ctx->stream, mask, imp, ctx->mbw,
                           ctx->mbh, ctx->cfg.connectivity, ctx->T, ctx->cfg.sort_policy, imp_in_lds, ctx->owner_id, ctx->raw,
                           ctx->pcount);
    }
    LAUNCHED();
    const int nblk = (total + 255) / 256;
    hipLaunchKernelGGL(k_plan_rank, dim3(min(512, (total + 15) / 16)), dim3(256), 0, ctx->stream, ctx->raw, ctx->pcount, ctx->sorted,
                       ctx->rank_of_id);
    LAUNCHED();
    hipLaunchKernelGGL(k_plan_place, dim3(1), dim3(64), (size_t)ctx->free_cap * 12, ctx->stream, ctx->sorted,
                       ctx->pcount, ctx->cfg.halo, ctx->cfg.bin_size, ctx->cfg.max_bins, ctx->free_cap, ctx->cfg.rotate,
                       box_pos);
    LAUNCHED();
    hipLaunchKernelGGL(k_plan_emit, dim3(nblk), dim3(256), 0, ctx->stream, ctx->sorted, box_pos, ctx->pcount,
                       list, n_sel, ctx->owner_id, ctx->rank_of_id, ctx->mbw, per, ctx->cfg.halo, boxes, places,
                       counts);
    LAUNCHED();
#undef LAUNCHED
    return RH_OK;
}
