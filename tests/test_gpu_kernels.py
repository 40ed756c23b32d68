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


# 16 x 16 tiles, channels in groups of 4 (and 4 outputs), the patch kernel up to 64 input channels
@pytest.mark.parametrize("net,shape", [
    (wl.Net("plain", 1, 3, 1, 0.1), (2, 3, 16)), (wl.Net("plain", 4, 3, 2, 0.1), (1, 16, 17)),
    (wl.Net("plain", 6, 3, 3, 0.1), (2, 15, 33)), (wl.Net("res", 16, 1, 2, 0.05), (3, 31, 32)),
    (wl.Net("edsr", 20, 1, 3, 0.05), (1, 17, 5)), (wl.Net("plain", 64, 3, 2, 0.1), (1, 18, 20)),
    (wl.Net("plain", 65, 3, 2, 0.1), (1, 18, 20)),
])
def test_fp32_conv_shapes(net, shape):
    N, H, W = shape
    blob = wl.make_weights(net, 11, "fp32")
    rh = RH(frame_w=64, frame_h=64, max_frames=1, halo=2, bin_size=32, max_bins=4, net=net, weights=blob, precision="fp32")
    x = np.random.default_rng(N * H * W).integers(0, 256, (N, H, W, 3), dtype=np.uint8)
    out = torch.full((N, H * net.scale, W * net.scale, 3), float("nan"), device="cuda")
    rh.enhance(dev(x), out=out)
    # the bar of the fp32 path (1e-5 of the norm, sums of at most 9 x 65 products)
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
# either neighbourhood; turned boxes; bins that run out in either loop
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
