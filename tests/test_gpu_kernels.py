"""Kernels at the sizes where they can go wrong: edges of tiles, remainders, both sides of every
line at which the dispatch changes kernels.  Reference: the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from paper_2407_16990_amd import RH
from test_gpu_parity import exact_border_check
from gpu_common import check_net, check_select_and_plan, dev, gpu_select, make_rh

pytestmark = pytest.mark.gpu


# 16 x 16 tiles, channels in groups of 4 (and 4 outputs), the patch kernel up to 120 input channels
@pytest.mark.parametrize("net,shape", [
    (wl.Net("plain", 1, 3, 1, 0.1), (2, 3, 16)), (wl.Net("plain", 4, 3, 2, 0.1), (1, 16, 17)),
    (wl.Net("plain", 6, 3, 3, 0.1), (2, 15, 33)), (wl.Net("res", 16, 1, 2, 0.05), (3, 31, 32)),
    (wl.Net("edsr", 20, 1, 3, 0.05), (1, 17, 5)), (wl.Net("plain", 64, 3, 2, 0.1), (1, 18, 20)),
    (wl.Net("plain", 65, 3, 2, 0.1), (1, 18, 20)), (wl.Net("res", 119, 1, 2, 0.05), (1, 17, 19)),
    (wl.Net("plain", 120, 3, 2, 0.1), (2, 18, 20)), (wl.Net("plain", 121, 3, 2, 0.1), (1, 18, 20)),
])
def test_fp32_conv_shapes(net, shape):
    N, H, W = shape
    blob = wl.make_weights(net, 11, "fp32")
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=blob, precision="fp32")
    x = np.random.default_rng(N * H * W).integers(0, 256, (N, H, W, 3), dtype=np.uint8)
    out = torch.full((N, H * net.scale, W * net.scale, 3), float("nan"), device="cuda")
    rh.enhance(dev(x), out=out)
    # the bar of the fp32 path (1e-5 of the norm, sums of at most 9 x 121 products)
    check_net(out.cpu().numpy(), oracle.sr_forward(net, blob, x), "fp32", f"{net} {shape}")
    rh.close()


# 32-channel nets: two convs per launch on tiles of 16 x 32; an odd number of plain layers leaves one over, an
# odd and an even number of residual blocks end in different buffers of the long skip
@pytest.mark.parametrize("net,shape", [
    (wl.Net("res", 32, 1, 2, 0.03), (2, 16, 32)), (wl.Net("res", 32, 2, 3, 0.03), (1, 17, 33)),
    (wl.Net("res", 32, 3, 1, 0.03), (1, 16, 16)), (wl.Net("plain", 32, 4, 2, 0.1), (1, 34, 31)),
    (wl.Net("plain", 32, 5, 2, 0.1), (2, 15, 66)), (wl.Net("plain", 32, 3, 2, 0.1), (1, 18, 36)),
    (wl.Net("edsr", 32, 1, 2, 0.03), (1, 33, 20)), (wl.Net("edsr", 32, 2, 4, 0.03), (1, 18, 40)),
])
def test_block32_shapes(net, shape):
    N, H, W = shape
    blob = wl.make_weights(net, 12, "bf16")
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=blob, precision="bf16")
    x = np.random.default_rng(H * W).integers(0, 256, (N, H, W, 3), dtype=np.uint8)
    out = torch.full((N, H * net.scale, W * net.scale, 3), float("nan"), device="cuda")
    rh.enhance(dev(x), out=out)
    check_net(out.cpu().numpy(), oracle.sr_forward(net, blob, x), "bf16", f"{net} {shape}")
    rh.close()


def test_block32_tiles_do_not_depend_on_the_batch():
    # more tiles than resident workgroups, whole and partial rounds, both tile directions, a device-side count
    net = wl.Net("res", 32, 3, 2, 0.03)
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=wl.make_weights(net, 13, "bf16"),
            precision="bf16")
    x = torch.randint(0, 256, (61, 80, 100, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    out = torch.full((61, 160, 200, 3), -1.0, device="cuda")
    rh.enhance(x, n=61, n_valid=torch.tensor([60], dtype=torch.int32, device="cuda"), out=out)
    one = torch.empty((1, 160, 200, 3), device="cuda")
    for i in (0, 1, 29, 58, 59):
        rh.enhance(x[i:i + 1].contiguous(), out=one)
        assert torch.equal(one[0], out[i]), i
    assert bool((out[60] == -1.0).all())
    rh.close()


# Plans whose list of free rectangles stays in one, grows to several, or outgrows the registers' chunks of 64
# (most entries: 32, 181, 206, 425, 263), of up to 16 frames (one launch) and more; isolated macroblocks with
# either neighbourhood; turned boxes; bins that run out
@pytest.mark.parametrize("F,w,h,halo,S,frac,kind,T,conn,rotate,max_bins", [
    (17, 480, 272, 10, 128, 0.5, "clustered", 0, 8, False, 400), (128, 480, 272, 10, 128, 0.2, "clustered", 0, 8, False, 800),
    (60, 480, 272, 10, 128, 0.12, "uniform", 0, 8, False, 600), (16, 640, 368, 10, 192, 0.4, "clustered", 3, 8, False, 300),
    (12, 1008, 560, 10, 128, 0.5, "clustered", 0, 8, False, 900), (16, 480, 272, 10, 128, 0.12, "uniform", 0, 4, True, 200),
    (60, 480, 272, 10, 128, 0.12, "uniform", 0, 4, True, 600), (16, 640, 368, 10, 192, 0.4, "clustered", 3, 8, True, 300),
    (16, 480, 272, 10, 128, 0.12, "uniform", 0, 8, False, 37), (60, 480, 272, 10, 128, 0.12, "uniform", 0, 8, False, 350),
    (20, 64, 1024, 0, 16, 0.3, "uniform", 0, 8, False, 2000), (1, 1024, 32, 3, 64, 1.0, "uniform", 2, 8, True, 60),
])
def test_plan_list_lengths(F, w, h, halo, S, frac, kind, T, conn, rotate, max_bins):
    cfg = wl.replace(wl.config(3), n_frames=F, width=w, height=h, importance=kind, frac=frac, halo=halo, bin_size=S)
    frames = np.random.default_rng(F).integers(0, 256, (F, h, w, 3), dtype=np.uint8)
    net = wl.Net("plain", 1, 2, 1)
    rh = make_rh(wl.replace(cfg, net=net), wl.make_weights(net, 0, "fp32"), max_bins=max_bins, precision="fp32", connectivity=conn,
                 max_box_mbs=T, rotate=rotate)
    plan, _, _ = check_select_and_plan(rh, cfg, frames, wl.make_importance(cfg), wl.make_segments(cfg), conn=conn, T=T or None,
                                       max_bins=max_bins, rotate=rotate)
    assert plan.overflow == (max_bins in (37, 350))
    rh.close()


# Selection: queues that are kept in registers (up to 16 384 keys) and longer ones, frames that belong to no segment
# before, between and after the segments, empty segments, more segments than one launch's arguments hold (64)
@pytest.mark.parametrize("F,w,h,segs,levels", [
    (32, 480, 272, [(0, 32, 3000)], 0), (33, 480, 272, [(0, 33, 16829)], 0), (128, 480, 272, [(1, 127, 13056)], 7),
    (40, 480, 272, [(2, 3, 1), (5, 5, 4), (9, 38, 14000)], 3), (64, 64, 16, [(i, i + 1, i % 6) for i in range(64)], 2),
    (70, 64, 16, [(i, i + 1, i % 6) for i in range(1, 66)], 2), (5, 64, 16, [], 0), (3, 16, 16, [(0, 3, 2)], 1),
])
@pytest.mark.parametrize("mode", ["topk", "threshold"])
def test_select_sizes(F, w, h, segs, levels, mode):
    cfg = wl.replace(wl.config(3), n_frames=F, width=w, height=h)
    r = np.random.default_rng(F)
    imp = r.standard_normal((F, h // 16, w // 16)).astype(np.float32)
    if levels:
        imp = np.round(imp * levels) / levels
    imp.reshape(-1)[::97] = np.nan
    net = wl.Net("plain", 1, 2, 1)
    rh = make_rh(wl.replace(cfg, net=net), wl.make_weights(net, 0, "fp32"), max_bins=4, precision="fp32")
    thr = [0.3 + 0.1 * (i % 5) for i in range(len(segs))] if mode == "threshold" else None
    o_mask, o_list = oracle.select(imp, np.array(segs, dtype=np.uint32).reshape(-1, 3), mode, thr)
    for _ in range(2):                                       # the second call finds the first one's tables
        g_mask, g_list, _ = gpu_select(rh, imp, [s + ((thr[i],) if thr else ()) for i, s in enumerate(segs)], mode)
        assert np.array_equal(g_mask, o_mask) and np.array_equal(g_list, o_list)
    rh.close()


# Boxes that fill a bin among others: numbered by groups of 64 while bins are left for a whole group, one by one behind that
# (bins that run out in a group's first, middle and last boxes, after one group and more); one and several chunks of the list
@pytest.mark.parametrize("F,S,T,max_bins", [(16, 128, 0, 200), (16, 128, 0, 63), (16, 128, 0, 64), (16, 128, 0, 66), (40, 128, 0, 400), (40, 128, 0, 129),
                                            (40, 128, 0, 190), (40, 96, 0, 600), (40, 96, 0, 260), (64, 128, 5, 700), (64, 192, 0, 300), (1, 128, 0, 80)])
@pytest.mark.parametrize("rotate", [False, True])
def test_plan_full_bins(F, S, T, max_bins, rotate):
    cfg = wl.replace(wl.config(3), n_frames=F, width=480, height=272, frac=0.35, halo=10, bin_size=S)
    frames = np.random.default_rng(F).integers(0, 256, (F, 272, 480, 3), dtype=np.uint8)
    net = wl.Net("plain", 1, 2, 1)
    rh = make_rh(wl.replace(cfg, net=net), wl.make_weights(net, 0, "fp32"), max_bins=max_bins, precision="fp32", max_box_mbs=T, rotate=rotate)
    check_select_and_plan(rh, cfg, frames, wl.make_importance(cfg), wl.make_segments(cfg), T=T or None, max_bins=max_bins, rotate=rotate)
    rh.close()


# The upsampler and last conv as one 5 x 5 conv: tiles of 8 x 32, rows and columns left over, images of hardly more than the ring,
# two and four waves that share a sum
@pytest.mark.parametrize("scale", [2, 3, 4])
@pytest.mark.parametrize("channels", [32, 64])
@pytest.mark.parametrize("shape", [(1, 5, 5), (2, 7, 31), (3, 8, 33), (1, 9, 64), (2, 17, 70)])
def test_fold_tiles(scale, channels, shape):
    N, H, W = shape
    net = wl.Net("edsr", channels, 1, scale, 0.02)
    blob = wl.make_weights(net, 12, "bf16")
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=blob, precision="bf16")
    x = np.random.default_rng(N * H * W).integers(0, 256, (N, H, W, 3), dtype=np.uint8)
    out = torch.full((N, H * scale, W * scale, 3), float("nan"), device="cuda")
    rh.enhance(dev(x), out=out)
    # the bar of the bf16 path; a tap, row or wave's share left out is several per cent
    check_net(out.cpu().numpy(), oracle.sr_forward(net, blob, x), "bf16", f"{net} {shape}")
    rh.close()


# Paste with one and with four input rows a wave, both sides of the line between them (5/8 scale^2 strips a compute unit),
# frames with cut macroblocks and row pitches of every alignment, turned boxes, floats of the pasted macroblocks
@pytest.mark.parametrize("scale,w,h", [(1, 160, 48), (2, 160, 112), (3, 160, 112), (4, 192, 112), (1, 157, 45), (2, 150, 101), (3, 147, 107), (4, 185, 99)])
@pytest.mark.parametrize("side", [0, 1])
def test_unpack_rows_per_wave(scale, w, h, side):
    mbw, mbh, nmb = -(-w // 16), -(-h // 16), 64 // (4 * scale)
    strips = -(-mbw // nmb) * mbh
    F = 5 * scale * scale * torch.cuda.get_device_properties(0).multi_processor_count // (8 * strips) + side
    cfg = wl.replace(wl.config(3), n_frames=F, width=w, height=h, importance="uniform", frac=0.08, halo=3, bin_size=96)
    r = np.random.default_rng(F)
    frames = r.integers(0, 256, (F, h, w, 3), dtype=np.uint8)
    net = wl.Net("plain", 16, 2, scale)
    most = F * mbw * mbh // 20 + 8
    rh = make_rh(wl.replace(cfg, net=net), wl.make_weights(net, 0, "fp32"), max_bins=most, precision="fp32", rotate=True)
    imp = r.random((F, mbh, mbw), dtype=np.float32)
    plan, po, (d_frames, _, _) = check_select_and_plan(rh, cfg, frames, imp, np.array([[0, F, F * mbw * mbh // 12]], dtype=np.uint32), max_bins=most, rotate=True)
    out = (0.2 * r.standard_normal((plan.n_bins, 96 * scale, 96 * scale, 3))).astype(np.float32)
    hr, sel = rh.unpack(torch.from_numpy(out).cuda(), po.places, po.counts[3:4], d_frames, want_sel=True)
    o_hr, o_sel = oracle.unpack(frames, scale, out, plan.places, place_rot=plan.place_rot)
    assert np.array_equal(hr.cpu().numpy(), o_hr)
    # in [0, 1]: one division and one addition in fp32 on both sides, a few units of 2^-24 at most
    assert np.abs(sel.cpu().numpy()[: len(plan.places)] - o_sel).max() <= 1e-6
    rh.close()


# Exact-border mode's pixel mask: sides that are not multiples of 32 (words and tiles cut), of 8, fewer than 32 pixels,
# both resolutions (the second upsampling conv of x4 runs on twice the mask's grid), turned boxes, every topology
@pytest.mark.parametrize("net,halo,S,rotate", [
    (wl.Net("edsr", 64, 1, 4, 0.02), 5, 76, True), (wl.Net("edsr", 64, 1, 2, 0.02), 7, 44, False),
    (wl.Net("edsr", 64, 1, 3, 0.02), 3, 100, True), (wl.Net("res", 64, 1, 2, 0.02), 6, 28, True),
    (wl.Net("plain", 64, 4, 2, 0.1), 4, 64, False), (wl.Net("edsr", 64, 1, 4, 0.02), 6, 36, False),
])
def test_exact_border_mask(net, halo, S, rotate):
    cfg = wl.replace(wl.config(3), n_frames=2, width=112, height=80, halo=halo, bin_size=S, net=net)
    exact_border_check(cfg, "bf16", rotate=rotate)


# Bins that run out in each of the first fit's three loops: by the first box that needs bin `max_bins`, the list holds
# about 31 rectangles (10 bins: one chunk of registers), 160 (40: several chunks), 385 (110: LDS), 400 (the last bin of 145 or
# 183); upright and turned; 16 frames are planned in one launch, 20 in several.  All boxes from that one on are
# without a bin, the ones before it keep theirs.
@pytest.mark.parametrize("F,max_bins", [(16, 10), (16, 40), (16, 110), (16, 144), (20, 10), (20, 40), (20, 110), (20, 182)])
@pytest.mark.parametrize("rotate", [False, True])
def test_plan_runs_out_of_bins_in_every_loop(F, max_bins, rotate):
    cfg = wl.replace(wl.config(3), n_frames=F, width=640, height=368, frac=0.4, halo=10, bin_size=192)
    frames = np.random.default_rng(F).integers(0, 256, (F, 368, 640, 3), dtype=np.uint8)
    net = wl.Net("plain", 1, 2, 1)
    rh = make_rh(wl.replace(cfg, net=net), wl.make_weights(net, 0, "fp32"), max_bins=max_bins, precision="fp32", max_box_mbs=3, rotate=rotate)
    plan, _, _ = check_select_and_plan(rh, cfg, frames, wl.make_importance(cfg), wl.make_segments(cfg), T=3, max_bins=max_bins, rotate=rotate)
    assert plan.overflow and plan.n_bins == max_bins
    rh.close()


# Networks of weights 0 and +-1 on images of 0 and 255: every product, sum and activation is a whole number of at most
# 256, which bf16 holds, so no order of sums and no rounding point is left that could differ, and the output has to
# be the oracle's in every bit - at every tile edge, padded border and cleared pixel.
def whole_number_weights(net, seed, taps):
    """`taps` weights of +-1 per output (the last conv: 40), biases 0 or 1."""
    r = np.random.default_rng(seed)
    parts, bound, layers = [], 1, wl.net_layers(net)
    for i, (cin, cout, role) in enumerate(layers):
        n = 40 if role == "last" else taps
        w = np.zeros((cout, 9 * cin), dtype=np.float32)
        at = np.argsort(r.random(w.shape), axis=1)[:, :min(n, 9 * cin)]
        np.put_along_axis(w, at, r.choice(np.float32([-1, 1]), at.shape), axis=1)
        parts += [w.ravel(), r.integers(0, 2, cout).astype(np.float32)]
        skipped = block_in if role == "res2" else head if net.topology == "edsr" and i == 2 * net.n_blocks + 1 else 0
        if role != "res2":
            block_in = bound
        bound = n * bound + 1 + skipped
        if i == 0:
            head = bound
        assert role == "last" or bound <= 256, (i, bound)
    return np.concatenate(parts)


WHOLE_NETS = [(wl.Net("res", 32, 2, 2), "bf16", 2), (wl.Net("res", 32, 3, 1), "bf16", 1), (wl.Net("plain", 32, 6, 2), "bf16", 2),
              (wl.Net("plain", 32, 7, 3), "bf16", 2), (wl.Net("edsr", 32, 1, 4), "bf16", 2), (wl.Net("edsr", 32, 2, 3), "bf16", 1),
              (wl.Net("res", 64, 2, 2), "bf16", 2), (wl.Net("plain", 64, 5, 2), "bf16", 2), (wl.Net("edsr", 64, 1, 2), "bf16", 2),
              (wl.Net("edsr", 64, 1, 3), "bf16", 2), (wl.Net("edsr", 64, 1, 4), "bf16", 2),
              (wl.Net("plain", 16, 4, 2), "fp32", 2), (wl.Net("edsr", 20, 1, 4), "fp32", 2), (wl.Net("res", 64, 2, 2), "fp32", 2)]


@pytest.mark.parametrize("net,precision,taps,tail", [c + (False,) for c in WHOLE_NETS] +
                         [c + (True,) for c in WHOLE_NETS if c[0].topology == "edsr" and c[1] == "bf16"])      # and layer by layer
@pytest.mark.parametrize("shape", [(2, 37, 70), (1, 16, 32), (3, 19, 33)])
def test_whole_number_nets_are_exact(net, precision, taps, tail, shape):
    N, H, W = shape
    blob = whole_number_weights(net, 3, taps)
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=blob, precision=precision, per_layer_tail=tail)
    x = np.random.default_rng(N * H * W).integers(0, 2, (N, H, W, 3), dtype=np.uint8) * np.uint8(255)
    out = torch.full((N, H * net.scale, W * net.scale, 3), float("nan"), device="cuda")
    rh.enhance(dev(x), out=out)
    o = oracle.sr_forward(net, blob, x)
    assert len(np.unique(o)) > 5 and np.array_equal(out.cpu().numpy().astype(np.float64), o)
    rh.close()


# Exact-border mode with boxes that leave the frame on all sides: the 64-channel convs' bit mask, k_zero_outside elsewhere
@pytest.mark.parametrize("net,precision,taps", WHOLE_NETS)
@pytest.mark.parametrize("halo,S,rotate", [(5, 76, True), (6, 44, False), (3, 100, True)])
def test_whole_number_nets_are_exact_at_frame_borders(net, precision, taps, halo, S, rotate):
    cfg = wl.replace(wl.config(3), n_frames=2, width=112, height=75, halo=halo, bin_size=S, net=net)
    frames = np.random.default_rng(S).integers(0, 2, (2, 75, 112, 3), dtype=np.uint8) * np.uint8(255)
    imp = wl.make_importance(cfg)
    imp[:, 0, :] += 5.0; imp[:, :, 0] += 5.0; imp[:, -1, -3:] += 5.0
    blob = whole_number_weights(net, 4, taps)
    rh = make_rh(cfg, blob, precision=precision, rotate=rotate)
    plan, po, (_, _, o_bins) = check_select_and_plan(rh, cfg, frames, imp, wl.make_segments(cfg), rotate=rotate)
    keep = oracle.border_keep(cfg.height, cfg.width, plan.boxes, halo, S, plan.n_bins)
    o = oracle.sr_forward(net, blob, o_bins, keep)
    out = torch.full((plan.n_bins, S * net.scale, S * net.scale, 3), float("nan"), device="cuda")
    rh.enhance_exact(po.bins, po.boxes, po.counts, n=plan.n_bins, n_valid=po.counts[1:2], out=out)
    assert (keep == 0).any() and not np.array_equal(o, oracle.sr_forward(net, blob, o_bins))
    assert np.array_equal(out.cpu().numpy().astype(np.float64), o)
    rh.close()


# Exact-border mode without boxes clears nothing and runs every layer in a launch of its own (32 channels), or with a mask
# that keeps every pixel (64): the same bits as the plain call's pairs of convs and plain stores.
@pytest.mark.parametrize("net", [wl.Net("res", 32, 3, 2, 0.03), wl.Net("plain", 32, 5, 2, 0.1), wl.Net("plain", 32, 6, 3, 0.1), wl.Net("edsr", 32, 2, 3, 0.03),
                                 wl.Net("res", 64, 2, 2, 0.02), wl.Net("plain", 64, 5, 2, 0.1), wl.Net("edsr", 64, 1, 2, 0.02),
                                 wl.Net("edsr", 64, 1, 3, 0.02), wl.Net("edsr", 64, 1, 4, 0.02)])
@pytest.mark.parametrize("S,N", [(36, 5), (100, 3), (64, 70)])
def test_exact_mode_without_boxes_is_the_plain_call_bit_for_bit(net, S, N):
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=S, max_bins=N, net=net, weights=wl.make_weights(net, 14, "bf16"),
            precision="bf16", per_layer_tail=True)
    x = torch.randint(0, 256, (N, S, S, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(S))
    boxes, counts = torch.zeros((1, 24), dtype=torch.uint8, device="cuda"), torch.zeros(4, dtype=torch.int32, device="cuda")
    assert torch.equal(rh.enhance(x), rh.enhance_exact(x, boxes, counts))
    rh.close()


# The patch kernel's sums go in the order of the kernel for more than 120 channels: a net in 124 channels whose added
# ones carry zeros gives the same bits (a product with zero leaves a sum as it is).
@pytest.mark.parametrize("net", [wl.Net("plain", 6, 4, 3, 0.1), wl.Net("res", 16, 2, 2, 0.05), wl.Net("edsr", 20, 1, 4, 0.05), wl.Net("edsr", 64, 1, 2, 0.05),
                                 wl.Net("plain", 65, 4, 2, 0.1), wl.Net("res", 119, 1, 2, 0.05), wl.Net("edsr", 120, 1, 2, 0.05)])
def test_fp32_patch_kernel_is_the_direct_kernel_bit_for_bit(net):
    big = wl.replace(net, channels=124)
    small_blob, parts, off = wl.make_weights(net, 15, "fp32"), [], 0
    for (ci, co, _), (cI, cO, _) in zip(wl.net_layers(net), wl.net_layers(big)):
        w, b = np.zeros((cO, 9, cI), dtype=np.float32), np.zeros(cO, dtype=np.float32)
        w[:co, :, :ci] = small_blob[off:off + co * 9 * ci].reshape(co, 9, ci); off += co * 9 * ci
        b[:co] = small_blob[off:off + co]; off += co
        parts += [w.ravel(), b]
    x = torch.randint(0, 256, (2, 35, 50, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    outs = []
    for n, blob in ((net, small_blob), (big, np.concatenate(parts))):
        rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=n, weights=blob, precision="fp32")
        outs.append(rh.enhance(x))
        rh.close()
    assert torch.equal(outs[0], outs[1])


# A step recorded into a graph after one eager step of the same size: nothing allocates, and every replay
# clears what it counts.  16 frames are planned in one launch, 20 in several.
@pytest.mark.parametrize("F,net", [(16, wl.Net("res", 64, 1, 2, 0.02)), (20, wl.Net("res", 32, 1, 2, 0.03)), (20, wl.Net("plain", 64, 3, 2, 0.1))])
def test_recorded_step_replays(F, net):
    cfg = wl.replace(wl.config(3), n_frames=F, width=160, height=112, halo=4, bin_size=64, net=net)
    blob, stream = wl.make_weights(net, 3, "bf16"), torch.cuda.Stream()
    frames, segs = dev(wl.make_frames(cfg)), [tuple(r) for r in wl.make_segments(cfg).tolist()]
    imps = [dev(np.roll(wl.make_importance(cfg), k, axis=0)) for k in range(4)]
    rh = make_rh(cfg, blob, max_bins=80, stream=stream)
    imp = imps[0].clone()
    po = None

    def step(po):
        po = rh.pack(frames, imp, *rh.select_regions(imp, segs), out=po)
        net_out = rh.enhance_exact(po.bins, po.boxes, po.counts, n=80, n_valid=po.counts[1:2])
        return po, rh.unpack(net_out, po.places, po.counts[3:4], frames)[0]

    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        po, _ = step(None)
        want = []
        for v in imps:
            imp.copy_(v)
            po, hr = step(po)
            want.append((po.counts.clone(), hr.clone()))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        _, hr = step(po)
    for k in (3, 0, 2, 1, 3):
        with torch.cuda.stream(stream):
            imp.copy_(imps[k])
            hr.zero_(); po.counts.zero_()
            graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(po.counts, want[k][0]) and torch.equal(hr, want[k][1]), k
    assert int(want[0][0][0]) > 0 and not torch.equal(want[0][1], want[1][1])
    rh.close()


def body_way(n, H, W):
    """How the body of a 64-channel net goes in the plain mode with no count: two layers a unit of so many rows, a layer at a time, or two convs or one a launch"""
    cu, cells = torch.cuda.get_device_properties(0).multi_processor_count, n * -(-H // 8) * -(-W // 32)
    rows = next((r for r in range(4, 23, 2) if n * -(-H // r) * -(-W // 30) <= cu), 0)
    if cells > (8 if W > 48 else 12) * cu:
        return "streams" if W > 48 else "launches"
    return f"{rows} rows" if rows else "few" if cells <= 4 * cu else "many"


# The body of a 64-channel net in one launch against the two convs or the conv a launch that larger batches take: the same images in a batch of that
# size with a device-side count.  Two layers a unit: one unit in all, fewer units than workgroups, ragged rows and columns.  A layer at a time, up
# to 4 units a workgroup and more: one and two and some rounds a layer, ragged rows and columns.  An odd number of layers, a first layer alone.
@pytest.mark.parametrize("net", [wl.Net("edsr", 64, 1, 2, 0.02), wl.Net("edsr", 64, 3, 4, 0.02), wl.Net("res", 64, 1, 2, 0.02), wl.Net("res", 64, 4, 3, 0.02),
                                 wl.Net("plain", 64, 4, 2, 0.1), wl.Net("plain", 64, 7, 2, 0.1)])
@pytest.mark.parametrize("n,H,W,way,other", [(1, 3, 5, "4 rows", "launches"), (1, 8, 32, "4 rows", "launches"), (2, 9, 33, "4 rows", "launches"), (3, 50, 100, "4 rows", "streams"),
                                             (7, 64, 128, "10 rows", "streams"), (31, 57, 33, "16 rows", "launches"), (9, 128, 128, "few", "streams"), (270, 8, 30, "few", "launches"),
                                             (130, 9, 33, "few", "launches"), (25, 57, 100, "few", "streams"), (40, 60, 140, "many", "streams"), (100, 50, 60, "many", "streams"),
                                             (2, 200, 1000, "many", "streams"), (150, 57, 40, "many", "launches")])
def test_one_launch_body_is_a_launch_per_layer_bit_for_bit(net, n, H, W, way, other):
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=wl.make_weights(net, 16, "bf16"),
            precision="bf16")
    lim = 12 * torch.cuda.get_device_properties(0).multi_processor_count
    cells = -(-H // 8) * -(-W // 32)
    assert n * cells <= lim
    big = lim // cells + 1
    assert (body_way(n, H, W), body_way(big, H, W)) == (way, other)
    x = torch.randint(0, 256, (n, H, W, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    xb = torch.zeros((big, H, W, 3), dtype=torch.uint8, device="cuda")
    xb[:n] = x
    count = torch.tensor([n], dtype=torch.int32, device="cuda")
    want = rh.enhance(xb, n_valid=count)[:n].clone()
    for _ in range(3):                                       # again with the counters of the call before
        assert torch.equal(rh.enhance(x), want)
    few = max(1, n // 2)
    got = rh.enhance(x, n_valid=torch.tensor([few], dtype=torch.int32, device="cuda"))
    assert torch.equal(got[:few], want[:few])
    assert torch.equal(rh.enhance(x, n_valid=torch.zeros(1, dtype=torch.int32, device="cuda"), out=got.fill_(3.0)), torch.full_like(got, 3.0))
    rh.close()


# Two contexts on two streams, each with units for every compute unit, a layer at a time or two layers a unit: whichever workgroups start, all units are done
@pytest.mark.parametrize("counts", [(40, 60), (28, 27), (28, 60)])
def test_one_launch_bodies_share_the_gpu(counts):
    net = wl.Net("edsr", 64, 4, 2, 0.02)
    rhs, xs, wants, streams = [], [], [], [torch.cuda.Stream(), torch.cuda.Stream()]
    for k in range(2):
        rhs.append(RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=64, max_bins=64, net=net, weights=wl.make_weights(net, 17 + k, "bf16"),
                      precision="bf16", stream=streams[k]))
        xs.append(torch.randint(0, 256, (counts[k], 64, 64, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(k)))
    outs = [[torch.zeros((len(x), 128, 128, 3), device="cuda") for _ in range(12)] for x in xs]
    torch.cuda.synchronize()
    for k in range(2):                                       # one alone
        wants.append(torch.zeros_like(outs[k][0]))
        torch.cuda.synchronize()
        rhs[k].enhance(xs[k], out=wants[k])
        torch.cuda.synchronize()
    for i in range(12):
        for k in range(2):
            rhs[k].enhance(xs[k], out=outs[k][i])
    torch.cuda.synchronize()
    for k in range(2):
        assert all(torch.equal(o, wants[k]) for o in outs[k])
        rhs[k].close()


# A small batch's body while another context's launches, two convs or one each, hold the compute units: workgroups of the body that find
# room only after its roll has closed leave, and the others do their share
@pytest.mark.parametrize("S,other", [(64, "streams"), (48, "launches")])
@pytest.mark.parametrize("n", [1, 12, 100])
def test_one_launch_body_beside_a_launch_per_layer(n, S, other):
    net = wl.Net("edsr", 64, 4, 2, 0.02)
    streams, counts = [torch.cuda.Stream(), torch.cuda.Stream()], [12 * torch.cuda.get_device_properties(0).multi_processor_count // (-(-S // 8) * -(-S // 32)) + 1, n]
    assert body_way(counts[0], S, S) == other and (body_way(n, S, S) == "many" if n == 100 else "rows" in body_way(n, S, S))
    rhs = [RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=64, max_bins=64, net=net, weights=wl.make_weights(net, 19, "bf16"),
              precision="bf16", stream=s) for s in streams]
    xs = [torch.randint(0, 256, (c, S, S, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(c)) for c in counts]
    wants, outs = [torch.zeros((c, 2 * S, 2 * S, 3), device="cuda") for c in counts], [torch.zeros((6, c, 2 * S, 2 * S, 3), device="cuda") for c in counts]
    for k in range(2):                                       # one alone
        torch.cuda.synchronize()
        rhs[k].enhance(xs[k], out=wants[k])
    torch.cuda.synchronize()
    for i in range(6):
        for k in range(2):
            rhs[k].enhance(xs[k], out=outs[k][i])
    torch.cuda.synchronize()
    for k in range(2):
        assert all(torch.equal(o, wants[k]) for o in outs[k])
        rhs[k].close()


# Two 64-channel convs a launch as streams of rows: strips of every number of 16-pixel tiles, one to many of them, images of three rows (the fewest that the
# library takes) and more rows than a workgroup's run.  Every image of a large batch as the same image in a small one, whose body is one launch of another kernel.
@pytest.mark.parametrize("net", [wl.Net("res", 64, 2, 2, 0.02), wl.Net("edsr", 64, 1, 3, 0.02), wl.Net("plain", 64, 5, 2, 0.1)])
@pytest.mark.parametrize("H,W", [(3, 49), (4, 64), (9, 56), (5, 80), (40, 96), (3, 112), (24, 128), (7, 129), (16, 160), (33, 192), (13, 333), (60, 480)])
def test_row_streams_are_the_one_launch_body_bit_for_bit(net, H, W):
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=wl.make_weights(net, 23, "bf16"),
            precision="bf16")
    cells = -(-H // 8) * -(-W // 32)
    big = 13 * torch.cuda.get_device_properties(0).multi_processor_count // cells + 1
    assert body_way(big, H, W) == "streams" and body_way(1, H, W) not in ("streams", "launches")
    x = torch.randint(0, 256, (5, H, W, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(W))
    want = torch.cat([rh.enhance(x[i:i + 1].clone()) for i in range(5)])
    xb = x[torch.arange(big, device="cuda") % 5].contiguous()
    got = rh.enhance(xb)
    for i in range(5):
        assert bool((got[i::5] == want[i]).all()), i
    some = torch.tensor([max(1, big // 3)], dtype=torch.int32, device="cuda")
    part = rh.enhance(xb, n_valid=some, out=torch.full_like(got, 3.0))
    assert torch.equal(part[:int(some)], got[:int(some)]) and bool((part[int(some):] == 3.0).all())
    rh.close()


# Room for 8 to 12 half tiles of 8 x 32 a compute unit: one launch for up to 5 valid ones, two convs a launch for more, whichever tensor either ends in.
# Nothing behind the count is written; after a call of the one, the other finds nothing of it.
@pytest.mark.parametrize("net", [wl.Net("edsr", 64, 2, 2, 0.02), wl.Net("edsr", 64, 3, 2, 0.02), wl.Net("res", 64, 1, 2, 0.02), wl.Net("res", 64, 4, 3, 0.02)]
                         + [wl.Net("plain", 64, k, 2, 0.1) for k in (4, 5, 6, 7, 8)])
@pytest.mark.parametrize("H,W", [(128, 128), (57, 97), (200, 500)])
def test_the_count_decides_between_one_launch_and_row_streams(net, H, W):
    cu, cells = torch.cuda.get_device_properties(0).multi_processor_count, -(-H // 8) * -(-W // 32)
    N, few = 10 * cu // cells, 5 * cu // cells
    assert 8 * cu < N * cells <= 12 * cu and few >= 1
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=wl.make_weights(net, 37, "bf16"), precision="bf16")
    x = torch.randint(0, 256, (N, H, W, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(H))
    want = rh.enhance(x)                                     # no count: row streams
    for k in (few, few + 1, 0, 1, N, few, N - 1):
        got = rh.enhance(x, n_valid=torch.tensor([k], dtype=torch.int32, device="cuda"), out=torch.full_like(want, 3.0))
        assert torch.equal(got[:k], want[:k]) and bool((got[k:] == 3.0).all()), k
    rh.close()


# A few images, two layers a unit of 4, 6, .. 22 rows of 30 pixels: the images end with a unit, a row or a pixel before or behind its end, and within it;
# an odd layer at the end; rows = 0: a unit too many.  Against the same images in a batch that goes two convs or one a launch.
def pair_shapes(rows, cu):
    def chosen(n, H, W):
        return next((r for r in range(4, 23, 2) if n * -(-H // r) * -(-W // 30) <= cu), 0)
    r = rows or 22
    for H, W in ((128, 128), (3 * r + 1, 91), (2 * r, 60), (4 * r - 1, 32), (r, 269), (r + 2, 31)):
        n = next((n for n in range(1, 2 * cu) if chosen(n, H, W) == rows), 0)
        if n:
            yield n, H, W


@pytest.mark.parametrize("net", [wl.Net("edsr", 64, 2, 2, 0.02), wl.Net("res", 64, 1, 2, 0.02), wl.Net("plain", 64, 4, 2, 0.1), wl.Net("plain", 64, 7, 2, 0.1)])
@pytest.mark.parametrize("rows", [4, 6, 8, 10, 12, 14, 16, 18, 20, 22, 0])
def test_two_layers_a_unit_are_the_larger_batch_bit_for_bit(net, rows):
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    shapes = list(pair_shapes(rows, cu))
    assert len(shapes) >= 2
    for n, H, W in shapes:
        rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=wl.make_weights(net, 29, "bf16"), precision="bf16")
        big = 12 * cu // (-(-H // 8) * -(-W // 32)) + 1
        x = torch.randint(0, 256, (n, H, W, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(n + H))
        xb = x[torch.arange(big, device="cuda") % n].contiguous()
        want = rh.enhance(xb)[:n].clone()
        for _ in range(3):                                   # again with the counters and buffers of the call before
            assert torch.equal(rh.enhance(x), want), (n, H, W)
        rh.close()


# The same in exact-border mode, whose convs clear what lies outside the frame, on 1 to 9 bins of a plan whose boxes leave the frame
@pytest.mark.parametrize("net", [wl.Net("edsr", 64, 1, 2, 0.02), wl.Net("plain", 64, 5, 2, 0.1)])
def test_two_layers_a_unit_at_frame_borders(net):
    cfg = wl.replace(wl.config(3), n_frames=16, width=240, height=139, halo=9, bin_size=128, net=net)
    imp = wl.make_importance(cfg)
    imp[:, 0, :] += 5.0; imp[:, :, 0] += 5.0; imp[:, -1, -3:] += 5.0
    most = 12 * torch.cuda.get_device_properties(0).multi_processor_count // 64 + 1
    rh = make_rh(cfg, wl.make_weights(net, 31, "bf16"), max_bins=most)
    segs = [tuple(r) for r in wl.make_segments(cfg).tolist()]
    d_imp = dev(imp)
    po = rh.pack(dev(wl.make_frames(cfg)), d_imp, *rh.select_regions(d_imp, segs))
    assert 9 <= int(po.counts[1]) <= most
    count = lambda k: torch.tensor([k], dtype=torch.int32, device="cuda")
    want = rh.enhance_exact(po.bins, po.boxes, po.counts, n=most, n_valid=count(9))[:9].clone()
    assert not torch.equal(want, rh.enhance(po.bins, n=9))
    for k in range(1, 10):
        got = rh.enhance_exact(po.bins, po.boxes, po.counts, n=9, n_valid=count(k))
        assert torch.equal(got[:k], want[:k]), k
    rh.close()


# fp32 convs with a device-side count, the patch requested ahead of it (up to 8 workgroups a compute unit) and behind it:
# the valid images as without a count, the others untouched, ragged tiles
@pytest.mark.parametrize("net", [wl.Net("plain", 16, 3, 2), wl.Net("res", 32, 1, 3), wl.Net("edsr", 16, 1, 2, 0.05), wl.Net("res", 24, 1, 2)])
@pytest.mark.parametrize("N,valid", [(1, 0), (3, 2), (5, 5), (400, 0), (400, 7), (400, 400)])
def test_fp32_images_behind_the_count(net, N, valid):
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=wl.make_weights(net, 5, "fp32"), precision="fp32")
    x = torch.randint(0, 256, (N, 37, 50, 3), dtype=torch.uint8, device="cuda", generator=torch.Generator("cuda").manual_seed(N + valid))
    want = torch.cat([rh.enhance(x[i:i + 1]) for i in range(min(N, 8))])
    out = torch.full((N, 37 * net.scale, 50 * net.scale, 3), 3.0, device="cuda")
    rh.enhance(x, out=out, n_valid=torch.tensor([valid], dtype=torch.int32, device="cuda"))
    k = min(valid, 8)
    assert torch.equal(out[:k], want[:k]) and bool((out[valid:] == 3.0).all()) and not bool((out[:valid] == 3.0).flatten(1).all(1).any())
    rh.close()
