"""What the C entry points do on the host: which kernels they launch in which order, what they
allocate, and how they end when a launch or an allocation fails.  A recording stand-in takes the
place of the HIP runtime (recording_hip.cpp), so this needs no GPU and runs no kernel; each test is a
child process, because the stand-in has to be loaded before librh.so."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = r'''
import ctypes as C, sys
rec = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
rec.rec_log.restype = C.c_char_p; rec.rec_new_left.restype = C.c_long; rec.rec_fail_new.argtypes = [C.c_long]
L.rh_last_error.restype = C.c_char_p
P = lambda n=1: C.c_void_p(n << 24)                      # stands for a device buffer
PLAIN, RES, EDSR = 0, 1, 2

def weights(top, ch, nb, s):
    io = [(3, ch)] + [(ch, ch)] * (nb - 2 if top == PLAIN else 2 * nb)
    if top == EDSR:
        io += [(ch, ch)] + ([(ch, ch * s * s)] if s < 4 else [(ch, 4 * ch)] * 2) + [(ch, 3)]
    else:
        io.append((ch, 3 * s * s))
    return (C.c_float * sum(9 * i * o + o for i, o in io))()

def create(top, ch, nb, s, bf16, w=480, h=272, F=32, halo=6, S=64, bins=8, tail=0):
    cfg = (C.c_int32 * 16)(w, h, F, halo, S, bins, 8, 0, bf16, top, ch, nb, s, 0, 0, tail)
    blob, ctx = weights(top, ch, nb, s), C.c_void_p()
    return L.rh_create(cfg, blob, C.c_size_t(len(blob)), None, C.byref(ctx)), ctx

def names(): return [n for n in rec.rec_log().decode().split("\n") if n]
def pack(ctx, F): return L.rh_pack(ctx, P(1), F, P(2), P(3), P(4), P(5), P(6), P(7), P(8), P(9))
'''


@pytest.fixture(scope="module")
def run_child(tmp_path_factory):
    from paper_2407_16990_amd import binding
    binding.load_library()                                   # built if it is missing or stale
    lib = str(tmp_path_factory.mktemp("rec") / "librecording_hip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "recording_hip.cpp")])

    def run(body):
        r = subprocess.run([sys.executable, "-c", PRELUDE + body + "\nprint('DONE')", lib, binding.lib_path()], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0 and r.stdout.strip().endswith("DONE"), r.stdout[-2000:] + r.stderr[-3000:]
    return run


@pytest.mark.parametrize("w,h,F", [(480, 272, 17), (480, 272, 32), (1040, 64, 2)])
def test_a_plan_does_not_depend_on_how_the_last_one_ended(run_child, w, h, F):
    """The labelling kernel appends boxes at a counter: whichever launch of the plan before was lost, and
    also where none was, the counter is cleared in the same call and ahead of everything that uses it."""
    run_child(f'''
st, ctx = create(PLAIN, 4, 2, 2, 0, w={w}, h={h}, F={F})
assert st == 0
def check():
    rec.rec_reset()
    assert pack(ctx, {F}) == 0
    n = names()
    assert "k_plan_zero" in n[0] and sum("k_plan_zero" in x for x in n) == 1, n
    return len(n)
launches = check()
for k in range(launches):
    rec.rec_reset(); rec.rec_fail_launch(k)
    assert pack(ctx, {F}) == 4, k                            # RH_E_DEVICE
    assert len(names()) == k                                 # and nothing behind the lost launch
    assert check() == launches
''')


@pytest.mark.parametrize("net", ["PLAIN, 64, 4, 2", "RES, 64, 1, 3", "EDSR, 64, 1, 4", "RES, 32, 1, 2"])
def test_an_exact_border_call_fits_the_workspace_of_an_equally_large_call(run_child, net):
    """rh_enhance on images of as many pixels, with the same layers, has sized the workspace: the exact-border call
    that follows neither allocates nor synchronises (it may be under stream capture)."""
    run_child(f'''
for S, shapes in ((36, [(6, 36, 36), (1, 36, 216), (81, 4, 24)]), (64, [(6, 64, 64), (2, 48, 256)]), (16, [(6, 16, 16)])):
    for n, h, w in shapes:
        st, ctx = create({net}, 1, halo=0, S=S, tail=1)
        assert st == 0 and n * h * w == 6 * S * S
        assert L.rh_enhance(ctx, P(1), n, h, w, P(2), None) == 0
        rec.rec_reset()
        assert L.rh_enhance_exact(ctx, P(1), 6, P(3), P(4), P(2), None) == 0
        assert (rec.rec_mallocs(), rec.rec_syncs()) == (0, 0), (S, n, h, w)
''')


def test_the_body_goes_in_one_launch_up_to_twelve_half_tiles_a_compute_unit(run_child):
    run_child('''
def bodies(call):
    rec.rec_reset()
    assert call() == 0
    return sum("k_conv_mfma_body" in x for x in names()), len(names())
for net, layers in ((EDSR, 64, 2, 4, 1), 5), ((RES, 64, 2, 2, 1), 4), ((PLAIN, 64, 6, 2, 1), 4):
    st, ctx = create(*net, S=128, bins=64)
    assert st == 0
    # half tiles of 8 x 32, 256 compute units; up to eight a unit where the other side is two convs a launch (widths above 48)
    for n, h, w in ((1, 3, 3), (32, 128, 128), (3072, 8, 32), (768, 9, 33)):
        assert bodies(lambda: L.rh_enhance(ctx, P(1), n, h, w, P(2), None)) == (1, 3), (net, n)
    for n, h, w in ((3073, 8, 32), (769, 9, 33)):
        assert bodies(lambda: L.rh_enhance(ctx, P(1), n, h, w, P(2), None)) == (0, layers + 2), (net, n)
    for n, h, w in ((33, 128, 128), (48, 128, 128), (49, 128, 128)):
        assert bodies(lambda: L.rh_enhance(ctx, P(1), n, h, w, P(2), None)) == (0, (layers + 1) // 2 + 2), (net, n)
    # between eight and twelve a device-side count decides: both are launched
    one, two = (1, 3), (0, (layers + 1) // 2 + 2)
    for n, h, w, want in ((32, 128, 128, one), (33, 128, 128, (1, two[1] + 1)), (48, 128, 128, (1, two[1] + 1)), (49, 128, 128, two), (2, 384, 768, (1, two[1] + 1)), (1, 520, 1024, two)):
        assert bodies(lambda: L.rh_enhance(ctx, P(1), n, h, w, P(2), P(7))) == want, (net, n)
    assert bodies(lambda: L.rh_enhance_exact(ctx, P(1), 48, P(3), P(4), P(2), None))[0] == 1
    assert bodies(lambda: L.rh_enhance_exact(ctx, P(1), 49, P(3), P(4), P(2), None))[0] == 0
    assert bodies(lambda: L.rh_enhance_masked(ctx, P(1), 3, P(3), P(4), P(2), None))[0] == 0
    if net[0] == EDSR:                                       # this mode goes in one launch where all images go two layers a unit of up to 22 x 30 pixels
        for n, one in ((3, 1), (8, 1), (9, 0), (33, 0)):
            assert bodies(lambda: L.rh_enhance_needed(ctx, P(1), n, P(3), P(4), P(2), None))[0] == one, n
''')


def test_a_call_of_as_many_pixels_fits_whatever_its_shape(run_child):
    """The workspace follows from a call's pixels: images of another shape, however ragged, neither allocate nor
    synchronise behind a call of as many or more pixels."""
    run_child('''
for net in ((EDSR, 64, 1, 4, 1), (PLAIN, 64, 5, 2, 1), (RES, 32, 1, 2, 1), (RES, 16, 1, 2, 0)):
    for px, shapes in ((64 * 64, [(455, 3, 3), (1, 4, 1024), (13, 9, 33), (1, 1024, 4)]), (40 * 128 * 128, [(40 * 64, 16, 16), (2206, 9, 33), (60000, 3, 3)])):
        st, ctx = create(*net)
        assert st == 0 and L.rh_enhance(ctx, P(1), 1, 128, px // 128, P(2), None) == 0
        for n, h, w in shapes:
            rec.rec_reset()
            assert n * h * w <= px and L.rh_enhance(ctx, P(1), n, h, w, P(2), None) == 0
            assert (rec.rec_mallocs(), rec.rec_syncs()) == (0, 0), (net, n, h, w)
''')


@pytest.mark.parametrize("net", ["PLAIN, 16, 3, 2, 0", "RES, 64, 1, 2, 1", "EDSR, 32, 1, 2, 1"])
def test_create_reports_any_failed_host_allocation(run_child, net):
    """Nothing throws across the C ABI: whichever host allocation fails, rh_create returns RH_E_NOMEM, with no context
    and nothing left on the device."""
    run_child(f'''
FAR = 1 << 40
rec.rec_fail_new(FAR)
st, ctx = create({net})
assert st == 0
total = FAR - rec.rec_new_left()
rec.rec_fail_new(-1)
L.rh_destroy(ctx)
assert rec.rec_live() == 0 and total > 8
for k in sorted(set(list(range(min(total, 40))) + [total * i // 40 for i in range(40)] + [total - 1])):
    rec.rec_fail_new(k)
    st, ctx = create({net})
    rec.rec_fail_new(-1)
    if st == 0:                                              # only a helper thread was not to be had: its share is done without it
        assert "{net}".startswith("EDSR")
        L.rh_destroy(ctx)
    else:
        assert st == 5 and not ctx.value, (k, total, st)     # RH_E_NOMEM
    assert rec.rec_live() == 0, k
''')


@pytest.mark.parametrize("net,modes", [("PLAIN, 32, 5, 2, 1", "plain exact"), ("RES, 32, 3, 2, 1", "plain exact"), ("EDSR, 32, 2, 3, 1", "plain exact"),
                                       ("RES, 64, 2, 2, 1", "plain exact masked needed"), ("EDSR, 64, 1, 4, 1", "plain exact masked needed"),
                                       ("EDSR, 8, 1, 4, 0", "plain exact"), ("PLAIN, 68, 3, 2, 0", "plain exact"), ("RES, 124, 1, 2, 0", "plain exact")])
@pytest.mark.parametrize("halo,tail", [(6, 0), (0, 1)])
def test_profile_counts_every_launch_once(run_child, net, modes, halo, tail):
    """rh_profile_read's counts add up to the kernels that went out, and those of the convs to the conv kernels."""
    run_child(f'''
st, ctx = create({net}, halo={halo}, tail={tail})
assert st == 0 and L.rh_profile_enable(ctx, 1) == 0
ms, n = (C.c_double * 8)(), (C.c_uint32 * 8)()
def counted(call):
    rec.rec_reset()
    st = call()
    if st == 7 and {tail}: return                            # the needed-region mode does not take a layer-by-layer tail
    assert st == 0, (st, L.rh_last_error(ctx))
    assert L.rh_profile_read(ctx, ms, n) == 0
    k = names()
    assert sum(n) == len(k), (list(n), k)
    convs = [x for x in k if any(s in x for s in ("k_conv_mfma", "k_block32", "k_conv3x3_f32", "k_conv_tail3", "k_conv_fold"))]
    cleared = [x for x in k if "k_zero_outside" in x]
    if convs:                                                # conv + last conv
        assert len(convs) <= n[4] + n[5] <= len(convs) + len(cleared) + 1, (list(n), k)
seg = (C.c_uint32 * 8)(0, 1, 3, 0, 1, 9, 5, 0)
counted(lambda: L.rh_select_regions(ctx, P(1), 9, seg, 2, 0, P(2), P(3), P(4)))
segs = (C.c_uint32 * (4 * 32))(*[v for i in range(32) for v in (i, i + 1, 1, 0)])
counted(lambda: L.rh_select_regions(ctx, P(1), 32, segs, 32, 0, P(2), P(3), P(4)))
for F in (1, 16, 17, 32): counted(lambda: pack(ctx, F))
for mode in "{modes}".split():
    for nv in (None, P(11)):
        counted({{"plain": lambda: L.rh_enhance(ctx, P(1), 5, 64, 64, P(2), nv),
                 "exact": lambda: L.rh_enhance_exact(ctx, P(1), 5, P(3), P(4), P(2), nv),
                 "masked": lambda: L.rh_enhance_masked(ctx, P(1), 5, P(3), P(4), P(2), nv),
                 "needed": lambda: L.rh_enhance_needed(ctx, P(1), 5, P(3), P(4), P(2), nv)}}[mode])
counted(lambda: L.rh_unpack(ctx, P(1), 5, 64, 64, P(2), P(3), P(4), 8, P(5), None))
''')


@pytest.mark.parametrize("channels,patch", [(64, True), (65, True), (120, True), (121, False)])
def test_fp32_convs_take_the_patch_kernel_as_long_as_the_patch_fits(run_child, channels, patch):
    run_child(f'''
st, ctx = create(RES, {channels}, 1, 2, 0)
assert st == 0
rec.rec_reset()
assert L.rh_enhance(ctx, P(1), 2, 20, 20, P(2), None) == 0
n = names()
assert len(n) == 4 and "k_conv3x3_f32_lds" in n[0], n        # the first conv has 3 input channels
assert all(("k_conv3x3_f32_lds" in x) == {patch} for x in n[1:]), n
''')


def test_fp32_convs_look_at_the_image_count_first_on_large_grids(run_child):
    """Images behind the count cost nothing but their empty workgroups: only a grid of at most 8 workgroups a compute
    unit requests its patches ahead of the count."""
    run_child('''
import re
for net, per in ((PLAIN, 16, 4, 2, 0), 16 * 4), ((RES, 32, 1, 2, 0), 16 * 8), ((RES, 24, 1, 2, 0), 16 * 6):      # per: workgroups an image
    st, ctx = create(*net)
    assert st == 0
    for n in (1, 8 * 256 // per, 8 * 256 // per + 1, 200):
        rec.rec_reset()
        assert L.rh_enhance(ctx, P(1), n, 64, 64, P(2), P(3)) == 0
        k = [re.search(r"k_conv3x3_f32_ldsILb[01]ELi([0-9]+)ELb([01])E", x).groups() for x in names()]
        assert k and all((ahead == "1") == (cin != "0" and per * n <= 8 * 256) for cin, ahead in k[:-1]), (net, n, k)
        if n == 200: assert all(ahead == "0" for _, ahead in k), k
''')


def test_profile_counts_every_launch_of_the_temporal_reuse(run_child):
    run_child('''
st, ctx = create(PLAIN, 4, 2, 2, 0, w=32, h=32, F=1030)
assert st == 0 and L.rh_profile_enable(ctx, 1) == 0
ms, n = (C.c_double * 8)(), (C.c_uint32 * 8)()
def counted(call):
    rec.rec_reset()
    assert call() == 0, L.rh_last_error(ctx)
    assert L.rh_profile_read(ctx, ms, n) == 0
    assert n[7] == sum(n) == len(names()), (list(n), names())
counted(lambda: L.rh_temporal_phi(ctx, P(1), 30, 12, 1, P(2)))
for ns in (1, 511, 512, 1024):
    off = (C.c_int32 * (ns + 1))(*range(ns + 1))
    counted(lambda: L.rh_temporal_select(ctx, P(1), off, ns, ns, P(2), P(3), P(4), P(5)))
counted(lambda: L.rh_temporal_spread(ctx, P(1), 30, P(2), P(3)))
''')


def test_a_wait_given_up_on_the_device_fails_the_next_call_once(run_child):
    run_child('''
rec.rec_pinned.restype = C.c_void_p
st, ctx = create(EDSR, 64, 1, 2, 1)
assert st == 0
lost = C.cast(rec.rec_pinned(), C.POINTER(C.c_uint32))
out = (C.c_uint32 * 4)()
calls = [lambda: L.rh_enhance(ctx, P(1), 5, 64, 64, P(2), None), lambda: L.rh_enhance_exact(ctx, P(1), 5, P(3), P(4), P(2), None),
         lambda: L.rh_enhance_masked(ctx, P(1), 5, P(3), P(4), P(2), None), lambda: L.rh_enhance_needed(ctx, P(1), 5, P(3), P(4), P(2), None),
         lambda: L.rh_read_counts(ctx, P(1), out)]
for call in calls:
    assert lost[0] == 0 and call() == 0
    lost[0] = 1
    rec.rec_reset()
    assert call() == 4 and not names() and b"undefined" in L.rh_last_error(ctx)     # RH_E_DEVICE, nothing launched
    assert call() == 0
L.rh_destroy(ctx)
assert rec.rec_live() == 0
for net in ((EDSR, 32, 1, 2, 1), (RES, 64, 1, 2, 0)):                        # no such launch: no such word
    st, ctx = create(*net)
    assert st == 0 and not rec.rec_pinned()
''')
