"""Who takes part in a launch of the one-launch body, and who leaves (csrc/conv_body_roll.h), on the CPU:
the numbers under which the units of a layer are dealt, for every number of workgroups at which the roll
can close, and for those that come after that - which must leave whatever the word holds by then."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "conv_body_roll.h"

static void need(bool ok, const char* what, unsigned grid, unsigned closes, unsigned units)
{
    if (!ok) { printf("%s: grid %u, closed at %u, %u units\n", what, grid, closes, units); exit(1); }
}

// `closes` workgroups sign, then (below the whole grid) one of them closes the roll and the others sign too late
static void run(unsigned grid, unsigned closes, unsigned units)
{
    std::vector<unsigned> sign(grid), took(grid, 0), order(grid);
    for (unsigned i = 0; i < grid; ++i) order[i] = (i * 7u + 3u) % grid;      // starting order of the workgroups: not their numbers
    if (grid % 7 == 0) for (unsigned i = 0; i < grid; ++i) order[i] = grid - 1 - i;
    uint32_t roll = 0;
    body_place p;
    for (unsigned i = 0; i < closes; ++i) {
        sign[i] = roll++;
        if (roll < grid) need(!body_roll_place(sign[i], roll, grid, order[i], &p), "decided too early", grid, closes, units);
    }
    if (closes < grid) {
        roll = body_roll_closed(roll);
        for (unsigned i = closes; i < grid; ++i) sign[i] = roll++;
    }
    const unsigned G = closes < units ? closes : units;
    for (unsigned i = 0; i < grid; ++i) {
        need(body_roll_place(sign[i], roll, grid, order[i], &p), "not decided", grid, closes, units);
        body_roll_spread(&p, grid, units);
        const bool leaves = body_roll_leaves(&p, units);
        if (i >= closes) { need(leaves, "a late workgroup stays", grid, closes, units); continue; }
        if (leaves) continue;
        need(p.G == G && p.wg < G, "number out of range", grid, closes, units);
        ++took[p.wg];
    }
    for (unsigned i = 0; i < G; ++i) need(took[i] == 1, "units without, or with two workgroups", grid, closes, units);
}

int main()
{
    for (unsigned grid : {1u, 2u, 3u, 7u, 16u, 24u, 32u, 255u, 256u, 304u})
        for (unsigned closes = 1; closes <= grid; ++closes)
            for (unsigned units : {0u, 1u, 2u, closes - 1, closes, closes + 1, grid, 4 * grid - 1, 4 * grid, 12 * grid, 1u << 20}) run(grid, closes, units);
    // the word as a late workgroup finds it: 100 had signed, and as many more came since
    body_place p;
    need(body_roll_place(0x80640064u, 0x80640065u, 256, 200, &p) && body_roll_leaves(&p, 640), "a late workgroup stays", 256, 100, 640);
    puts("ROLL_OK");
}
'''


def test_every_workgroup_on_the_roll_has_its_number_and_late_ones_leave(tmp_path):
    src, exe = str(tmp_path / "roll.cpp"), str(tmp_path / "roll")
    with open(src, "w") as f:
        f.write(PROGRAM)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                           "-I" + os.path.join(ROOT, "paper_2407_16990_amd", "csrc"), "-o", exe, src])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "ROLL_OK" in r.stdout, r.stdout + r.stderr
