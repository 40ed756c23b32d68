"""Kernels at the sizes where they can go wrong: edges of tiles, remainders, both sides of every
line at which the dispatch changes kernels.  Reference: the CPU oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from paper_2407_16990_amd import RH
from gpu_common import check_net, dev

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
