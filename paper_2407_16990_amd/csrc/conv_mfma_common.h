// Definitions shared by the MFMA convolution kernels (conv_mfma.hip, conv_mfma_duo.hip).
#pragma once
#include "rh_internal.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;

struct conv_args {
    const __bf16* in;        // [N][H][W][CIN]
    const uint4* wp;         // packed weights of this layer
    const float* bias;       // packed order
    void* out;
    const __bf16* skip;      // same shape as out, or null
    const uint32_t* n_valid;
    int N, H, W;
    int relu, ps, n_chunks;  // bf16 output mode
    int cout_real, s_final;  // fp32 output mode
    int rev;                 // 1: walk the tiles from the last to the first (k_conv_mfma_duo)
    // box-masked mode (k_conv_mfma_duo): only the half tiles (8 rows x 32 pixels) listed are computed.
    // tile_list: RH_CELL_ENTRY(n, cy, tx) in any order, cy counting rows of 8; n_list: their number
    // (both dev); null: all tiles
    const uint32_t* tile_list;
    const uint32_t* n_list;
    // exact-border mode (k_conv_mfma_duo): one bit per pixel, [N][H >> keep_sh][words of 32 pixels of W >> keep_sh], or null;
    // keep_sh: log2 of the output pixel grid's resolution over the mask's (before the pixel shuffle)
    const uint32_t* keep;
    int keep_sh;
};

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b)
{
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
    f32x2 v = {a, b};
    bf16x2 r = __builtin_convertvector(v, bf16x2);     // round to nearest even
    return *(uint32_t*)&r;
}

// ReLU of two packed bf16 values: a negative float has its sign bit set, i.e. is a negative
// 16-bit integer, and max(x, 0) on the integers leaves the others unchanged (-0 becomes +0).
// One packed instruction per pair, against two v_max_f32 per value for fmaxf on the fp32 inputs
// (the compiler adds a canonicalising max, also when the ReLU is written as a median of three).
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t u)
{
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    const s16x2 z = {0, 0};
    const s16x2 r = __builtin_elementwise_max(*(const s16x2*)&u, z);
    return *(const uint32_t*)&r;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every
// outstanding global load and store of the wave, which would expose the latency of the patch
// prefetch, the skip reads and the output stores once per tile.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

// Copies to LDS in inline asm set m0 and say so, for the compiler sets it too (lds_dma), and would otherwise take it for what it was before.  The compiler
// warns of a register that it does not keep for others; nothing is kept there.
#pragma clang diagnostic ignored "-Winline-asm"

// `bytes` from `src` to LDS, 16 bytes per thread and turn, with no registers between: every piece of a layer's
// weights is in flight at once.  `wave` (scalar) is the thread's wave of the THREADS / 64; the data is there
// after lds_dma_wait() of all waves and a barrier.
template <int THREADS, int BYTES>
__device__ __forceinline__ void lds_dma(uint8_t* lds, const void* src, int wave, int lane)
{
    static_assert(BYTES % 1024 == 0, "whole waves only");
#pragma unroll
    for (int i = 0; i < (BYTES + THREADS * 16 - 1) / (THREADS * 16); ++i) {
        const int off = (i * (THREADS / 64) + wave) * 1024;
        if ((i + 1) * THREADS * 16 > BYTES && off >= BYTES) break;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)((const uint8_t*)src + off + lane * 16),
                                         (__attribute__((address_space(3))) void*)(lds + off), 16, 0, 0);
    }
}
// The builtin (vmcnt 0, the other counters open), not inline asm: the compiler's own count of outstanding loads has to see it.
__device__ __forceinline__ void lds_dma_wait() { __builtin_amdgcn_s_waitcnt(0x0F70); asm volatile("" ::: "memory"); }

#define RSRC_FLAGS 0x00020000            // raw buffer, 32-bit data format (gfx9 family)
#define OOB_OFF 0x80000000u              // beyond any descriptor used here (images are < 2 GiB)
// Cache policy of a conv's output stores: written through the L2 (sc1) as they are made.  What stays dirty in the eight
// L2s is written back when the launch ends, before the next one may start, and a conv never reads its output again:
// 33 body convs on 3 bins of 128 x 128 484 -> 461 us per step, on 76 bins 2923 -> 2870, on 15 of 160 x 160 1197 -> 1164.
#define ST_THROUGH 16

// all 64-channel convs between the first one and the tail in one launch (conv_body.hip)
struct body_args {
    __bf16 *h, *a, *t;       // [N][H][W][64]: the first conv's output, and what the blocks are computed in
    const uint4* wp;         // the layers' packed weights, one behind the other
    const float* bias;       // 64 a layer
    const uint32_t* n_valid;
    const uint32_t* keep;    // as in conv_args, or null
    int N, H, W, layers, topology;
    uint32_t* roll;          // workgroups that take part; zero at the launch, as
    uint32_t* done;          // a layer at a time: [half tiles of 8 x 32][4], layers that each wave of its team has stored; two layers a unit:
                             // [units][BODY_PAIR_WORDS], of which the first says how many steps of two layers the unit has done
    uint32_t* lost;          // host memory: set to 1 where a wait was given up
    uint32_t img_magic, row_magic;       // division by the half tiles of an image and of its rows (set by the launcher)
};
// words for `roll` and `done` together; `done` begins BODY_ROLL_WORDS behind `roll`.  Two of those between are counts of images, written by the first
// conv's launch: the valid ones where they are so few that they go in one launch, else 0, and the valid ones where they are more, else 0.
#define BODY_ROLL_WORDS 32
#define BODY_FEW_WORD 8
#define BODY_MANY_WORD 9
#define BODY_MOST_CELLS 12               // half tiles of 8 x 32 a compute unit, at most: so much room `done` has
#define BODY_PAIR_WORDS 32               // of `done`, one unit of two layers (at most one a compute unit): a line each
static_assert(BODY_PAIR_WORDS <= 4 * BODY_MOST_CELLS, "the words of either way have room");
hipError_t rh_launch_conv_body(hipStream_t stream, int device, int n_cu, body_args a);
bool rh_conv_body_pairs(int n_cu, int N, int H, int W);        // all N images go two layers a unit (conv_body_pairs.h)
// two-team kernel for the 64-channel bf16-output convs (conv_mfma_duo.hip)
hipError_t rh_launch_conv_duo(hipStream_t stream, int device, const conv_args& a, int grid, bool skip, bool relu);
// two 3x3 convs of a 32-channel net in one launch (conv_block32.hip); res: a residual block, else two ReLU layers.  in != out
hipError_t rh_launch_block32(rh_ctx* ctx, const rh_layer& L1, const rh_layer& L2, const __bf16* in, __bf16* out, int N, int H, int W,
                             bool res, const uint32_t* n_valid);
// the same for 64 channels (conv_block64.hip); rh_block64_strips: how it cuts a width, false for those that it is not made for
bool rh_block64_strips(int W, int* strips, int* wo, int* tiles, int* tiles2);
hipError_t rh_launch_block64(rh_ctx* ctx, const rh_layer& L1, const rh_layer& L2, const __bf16* in, __bf16* out, int N, int H, int W,
                             bool res, const uint32_t* n_valid);
// last conv with 3 output channels and no pixel shuffle (conv_tail.hip)
hipError_t rh_launch_conv_tail3(hipStream_t stream, int device, const conv_args& a, int cin);
// first conv 3 -> C on the matrix cores (conv_head.hip)
hipError_t rh_launch_head_mfma(hipStream_t stream, int C, const uint8_t* in, const uint4* wp, const float* bias, __bf16* out,
                               int N, int H, int W, int relu, const uint32_t* n_valid, uint32_t* clear, uint32_t n_clear, int few);
// upsampler + last conv of an EDSR-shaped net as one composed 5 x 5 conv (conv_fold.hip): t -> raw network output
// tile_list / n_list (dev, or null for all tiles): the 8 x 32 tiles to compute, as RH_CELL_ENTRY(n, ty, tx)
rh_status rh_launch_fold(rh_ctx* ctx, const __bf16* t, float* out, int N, int H, int W, const uint32_t* n_valid, int rev,
                         const uint32_t* tile_list, const uint32_t* n_list);
