// Who takes part in a launch of k_conv_mfma_body: the arithmetic of its roll, for the kernel and for a host program.
//
// The roll is one word, zero at the launch.  While it is open it counts the workgroups that have signed; closed, it holds
// BODY_CLOSED, the number that had signed until then (15 bits) and, below, a count of those that came later.  It closes once
// and never again opens; a roll that all have signed stays open for good, since nobody closes that one.
#pragma once
#include <stdint.h>

#ifdef __HIP__
#include <hip/hip_runtime.h>
#define BODY_HD __host__ __device__ __forceinline__
#else
#define BODY_HD inline
#endif

#define BODY_CLOSED 0x80000000u

struct body_place { uint32_t wg, G; };       // number wg of the G workgroups among which the units are dealt

BODY_HD uint32_t body_roll_closed(uint32_t open) { return BODY_CLOSED | open << 16; }

// What the workgroup that found `sign` when it signed makes of the roll, which reads r now.  False: not decided yet, look again.
// G = 0: it came too late and takes no part.
BODY_HD bool body_roll_place(uint32_t sign, uint32_t r, uint32_t grid, uint32_t block, body_place* p)
{
    p->wg = 0; p->G = 0;
    if (sign & BODY_CLOSED) return true;
    if (r & BODY_CLOSED) { p->wg = sign; p->G = r >> 16 & 0x7FFFu; return true; }
    if (r == grid) { p->wg = block; p->G = grid; return true; }
    return false;
}

// Workgroups go to the 8 XCDs round-robin.  With many units in a layer an XCD takes a run of neighbouring ones; with few,
// pairs: in runs the XCDs work, in step, at addresses a power of two apart, on the same memory channels (EDSR x4 on
// 128 x 128 bins, us, runs / pairs: 4 bins 477 / 327, 8: 485 / 420; level on 16; on 15 bins of 160 x 160 958 / 967).
// The full roll only: who signs an early closed one is not known by its place on the chip.
BODY_HD void body_roll_spread(body_place* p, uint32_t grid, uint32_t layer_units)
{
    if (p->G != grid || p->G % 16) return;
    const uint32_t run = layer_units >= 4 * p->G ? p->G / 8 : 2, local = p->wg / 8;
    p->wg = local / run * (8 * run) + p->wg % 8 * run + local % run;
}

// A layer of fewer units than workgroups needs no more than one each; true: this workgroup has none, or takes no part.
BODY_HD bool body_roll_leaves(body_place* p, uint32_t layer_units)
{
    if (p->G > layer_units) p->G = layer_units;
    return p->wg >= p->G;
}
