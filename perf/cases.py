"""The work whose speed counts: the calls that a user of the region-aware enhancer makes, over the
range in which they are made, as cases with inputs, one pass, and what a pass cannot do without.

Kinds of case
  step      one batch through the whole path: select_regions -> pack -> enhance -> unpack
            (`mode` says which enhance: plain, needed, masked, exact)
  frames    the frame-based run: every frame enhanced whole, every macroblock pasted
  plan      select_regions -> pack only (a planner that tries geometries, or a batch prepared ahead)
  paste     unpack only, on network output that is at hand
  temporal  the temporal reuse of importance maps over a chunk of frames, run ahead of the path

Sizes are the benchmark configurations' (workloads/), the tests' and 360p-class streams'.
"""
import math
import random

import numpy as np
import torch

import workloads as wl
from paper_2407_16990_amd import RH
from paper_2407_16990_amd.binding import PackOut

MB = 16

_BASE = {"kind": "step", "mode": "plain", "precision": "bf16", "topology": "edsr", "channels": 64, "blocks": 16, "scale": 4,
         "frames": 16, "width": 480, "height": 272, "halo": 10, "bin": 128, "frac": 0.2, "importance": "clustered",
         "streams": 1, "rotate": False}


def _case(name, **kw):
    c = dict(_BASE, **kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a thumbnail-sized frame through a small fp32 net: nothing but latency and launches
        _case("step_fp32_1x320x192", precision="fp32", topology="plain", channels=16, blocks=4, scale=2, frames=1, width=320,
              height=192, halo=4, bin=64, frac=0.25),
        # one 360p frame of one live stream as it arrives (ragged height, the paper's 3-pixel halo)
        _case("step_edsr_x3_1x640x360", scale=3, frames=1, width=640, height=360, halo=3, frac=0.1),
        # a 32-channel residual net on eight frames: the memory-bound net
        _case("step_res32_x2_8x640x368", topology="res", channels=32, blocks=8, scale=2, frames=8, width=640, height=368, halo=6,
              bin=96, frac=0.3),
        # the headline batch: EDSR-baseline x4, a fifth of the macroblocks
        _case("step_edsr_x4_16x480x272"),
        # the same batch with isolated macroblocks: the most boxes per selected macroblock
        _case("step_scattered_x4_16x480x272", frac=0.1, importance="scattered"),
        # eight streams with budgets of their own in one batch: the largest step
        _case("step_edsr_x3_32x640x368", scale=3, frames=32, width=640, height=368, streams=8, frac=0.25, importance="heavy"),
        # the headline batch where only pasted pixels count
        _case("needed_edsr_x4_16x480x272", mode="needed"),
        # whole ragged frames' borders exact, boxes turned where that fits, odd frame count
        _case("exact_edsr_x2_5x630x355", mode="exact", scale=2, frames=5, width=630, height=355, halo=7, bin=160, frac=0.15, rotate=True),
        # every frame enhanced whole: what the region-based step is compared with
        _case("frames_edsr_x4_16x480x272", kind="frames", frac=1.0),
        # selection and stitching of eight batches at once
        _case("plan_128x480x272", kind="plan", precision="fp32", topology="plain", channels=16, blocks=2, frames=128),
        # pasting eight batches at once
        _case("paste_x4_128x480x272", kind="paste", precision="fp32", topology="plain", channels=16, blocks=2, frames=128),
        # a second of ten streams through the temporal reuse
        _case("temporal_10x30x480x272", kind="temporal", precision="fp32", topology="plain", channels=16, blocks=2, frames=300, streams=10),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _most_bins(c):
    """Bins that one plan can hold (its list of free rectangles is bounded)."""
    return 11000 // (c["bin"] // (MB + 2 * c["halo"])) ** 2


def draw(rng: random.Random):
    most = max(w["flops"] for w in map(work, listed()))
    while True:
        kind = rng.choice(["step"] * 6 + ["frames", "plan", "paste", "temporal"])
        c = _case(None, kind=kind, width=rng.randint(160, 680), height=rng.randint(112, 400),
                  importance=rng.choice(["clustered", "clustered", "heavy", "scattered"]), frac=round(rng.uniform(0.05, 0.5), 3),
                  halo=rng.randint(3, 12), bin=4 * rng.randint(24, 48), rotate=rng.random() < 0.2, scale=rng.choice([2, 3, 4]),
                  frames=_log(rng, 1, 32))
        if c["importance"] == "scattered":
            c["frac"] = round(c["frac"] / 4, 3)
        if rng.random() < 0.4:      # the benchmark's own bins
            c["bin"] = rng.choice([96, 128, 128, 192])
        if kind == "step" and rng.random() < 0.15:      # the fp32 path, on small nets
            c.update(precision="fp32", topology=rng.choice(["plain", "res"]), channels=16, blocks=rng.randint(2, 5), frames=rng.randint(1, 2),
                     width=rng.randint(160, 400), height=rng.randint(112, 240))
        elif kind in ("step", "frames"):
            top = rng.choice(["edsr", "edsr", "edsr", "res", "plain"])
            c.update(topology=top, channels=rng.choice([64, 64, 64, 32]), blocks=rng.choice([4, 8, 16, 16]))
            if kind == "step" and c["channels"] == 64:
                c["mode"] = rng.choice(["plain", "plain", "plain", "needed", "masked", "exact"])
        else:
            c.update(precision="fp32", topology="plain", channels=16, blocks=2)
            c["frames"] = _log(rng, 16, 300 if kind == "temporal" else 128)
        if kind == "frames":
            c["frac"] = 1.0
            c["frames"] = _log(rng, 1, 16)
        c["streams"] = rng.choice([s for s in (1, 2, 3, 4, 8, 10) if s <= c["frames"] and c["frames"] % s == 0])
        if work(c)["flops"] <= 0.9 * most and 1.6 * packed_pixels(c) / c["bin"] ** 2 + 16 <= _most_bins(c):
            return c


# ---------------------------------------------------------------------------------------------
# inputs, made on the GPU

def _frames(c, g):
    """u8 [F,H,W,3]: half noise, half three smooth blobs (the recipe of workloads.make_frames)."""
    F, H, W = c["frames"], c["height"], c["width"]
    yy = torch.arange(H, device="cuda", dtype=torch.float32).view(1, H, 1)
    xx = torch.arange(W, device="cuda", dtype=torch.float32).view(1, 1, W)
    out = torch.empty((F, H, W, 3), dtype=torch.uint8, device="cuda")
    for f0 in range(0, F, 32):
        n = min(32, F - f0)
        img = 0.5 * torch.randint(0, 256, (n, H, W, 3), generator=g, device="cuda").float()
        for _ in range(3):
            u = torch.rand((6, n, 1, 1), generator=g, device="cuda")
            sig = (0.1 + 0.2 * u[2]) * min(W, H)
            b = torch.exp(-((xx - u[0] * W) ** 2 + (yy - u[1] * H) ** 2) / (2 * sig * sig))
            img += 127.5 * b.unsqueeze(3) * (0.3 + 0.7 * u[3:6]).permute(1, 2, 3, 0)
        out[f0:f0 + n] = img.round_().clamp_(0, 255).to(torch.uint8)
    return out


def _importance(c, g):
    """f32 [F,MBH,MBW]: 1 to 4 blobs a frame (`heavy`: lognormal amplitudes) + noise, or independent values."""
    F, mbh, mbw = c["frames"], (c["height"] + 15) // 16, (c["width"] + 15) // 16
    if c["importance"] == "scattered":
        return torch.rand((F, mbh, mbw), generator=g, device="cuda")
    yy = torch.arange(mbh, device="cuda", dtype=torch.float32).view(1, mbh, 1)
    xx = torch.arange(mbw, device="cuda", dtype=torch.float32).view(1, 1, mbw)
    imp = 0.1 * torch.rand((F, mbh, mbw), generator=g, device="cuda")
    count = torch.randint(1, 5, (F, 1, 1), generator=g, device="cuda") if c["importance"] == "heavy" else 3
    for j in range(4):
        u = torch.rand((3, F, 1, 1), generator=g, device="cuda")
        amp = torch.randn((F, 1, 1), generator=g, device="cuda").exp() if c["importance"] == "heavy" else torch.ones((F, 1, 1), device="cuda")
        amp = amp * (j < count) if torch.is_tensor(count) else amp * float(j < count)
        sig = 2.0 + 4.0 * u[2]
        imp += amp * torch.exp(-((xx - u[0] * mbw) ** 2 + (yy - u[1] * mbh) ** 2) / (2 * sig * sig))
    return imp.contiguous()


def _residuals(c, g, r):
    """i16 [F,H,W]: coding noise, drifting objects, now and then a change of a quarter of the picture, and a
    few isolated pixels (the recipe of workloads.make_residuals)."""
    F, H, W = c["frames"], c["height"], c["width"]
    res = (3.0 * torch.randn((F, H, W), generator=g, device="cuda")).round_().to(torch.int16)
    hot = torch.randint(0, H * W, (F, 15), generator=g, device="cuda")
    res.view(F, -1).scatter_add_(1, hot, torch.full_like(hot, 60, dtype=torch.int16))
    tex = (torch.rand((41, 41), generator=g, device="cuda") < 0.85).to(torch.int16)
    per = F // c["streams"]
    for s in range(c["streams"]):
        objs = [[r.uniform(0, W), r.uniform(0, H), r.gauss(0, 4), r.gauss(0, 4), r.randint(3, 40), r.randint(3, 40), r.random() < 0.7]
                for _ in range(r.randint(2, 8))]
        for t in range(per):
            f = s * per + t
            for o in objs:
                o[0], o[1] = (o[0] + o[2]) % W, (o[1] + o[3]) % H
                o[6] = o[6] != (r.random() < 0.08)
                if o[6]:
                    x, y = int(o[0]), int(o[1])
                    w, h = min(o[4], W - x), min(o[5], H - y)
                    res[f, y:y + h, x:x + w] += tex[:h, :w] * (r.randint(25, 89) * r.choice((-1, 1)))
            if r.random() < 0.05:
                y, x = r.randrange(max(1, H // 2)), r.randrange(max(1, W // 2))
                res[f, y:y + H // 2, x:x + W // 2] += r.randint(30, 69)
    return res.clamp_(-255, 255)


def _segments(c, r):
    """Rows (first frame, end, k): one queue for the batch, or one for each stream with a budget of its own."""
    per, F, S = ((c["height"] + 15) // 16) * ((c["width"] + 15) // 16), c["frames"], c["streams"]
    if S == 1:
        return [(0, F, max(1, int(c["frac"] * F * per)))]
    n = F // S
    return [(s * n, (s + 1) * n, max(1, int(c["frac"] * r.uniform(0.4, 1.6) * n * per) if c["frac"] < 0.6 else int(c["frac"] * n * per))) for s in range(S)]


def _net(c):
    tail = {"edsr": 0.0125, "res": 0.03, "plain": 0.1}[c["topology"]]
    return wl.Net(c["topology"], c["channels"], c["blocks"], c["scale"], tail_scale=tail)


def prepare(case, seed):
    c, r = case, random.Random(seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    F, s, S = c["frames"], c["scale"], c["bin"]
    mbs = F * ((c["height"] + 15) // 16) * ((c["width"] + 15) // 16)
    net = _net(c)
    max_bins = min(_most_bins(c), max(16, 2 * int(packed_pixels(c) / (S * S)) + 2 * F + 32))
    rh = RH(frame_w=c["width"], frame_h=c["height"], max_frames=F, halo=c["halo"], bin_size=S, max_bins=max_bins, net=net,
            weights=wl.make_weights(net, seed, c["precision"]),
            precision=c["precision"], rotate=c["rotate"])
    st = {"case": c, "rh": rh}
    if c["kind"] == "temporal":
        st.update(res=_residuals(c, g, r), imp=_importance(c, g), off=[i * (F // c["streams"]) for i in range(c["streams"] + 1)],
                  total=max(c["streams"], F // 5))
        return st
    st["frames"] = _frames(c, g)
    if c["kind"] in ("step", "plan", "paste"):
        st["imp"], st["segs"] = _importance(c, g), _segments(c, r)
        st["po"] = PackOut(torch.zeros((max_bins, S, S, 3), dtype=torch.uint8, device="cuda"),
                           torch.zeros((mbs, 24), dtype=torch.uint8, device="cuda"),
                           torch.zeros((mbs, 16), dtype=torch.uint8, device="cuda"),
                           torch.zeros(4, dtype=torch.int32, device="cuda"))
    # the output buffers of a stream of such batches are sized once, by what they pack into and a quarter more
    st["cap"] = min(max_bins, int(1.25 * packed_pixels(c) / (S * S)) + F // 4 + 8)
    if c["kind"] == "paste":
        rh.pack(st["frames"], st["imp"], *rh.select_regions(st["imp"], st["segs"]), out=st["po"])
    if c["kind"] == "step":
        st["net_out"] = torch.zeros((st["cap"], S * s, S * s, 3), dtype=torch.float32, device="cuda")
    elif c["kind"] == "paste":
        st["net_out"] = 0.05 * torch.randn((st["cap"], S * s, S * s, 3), generator=g, device="cuda")
    elif c["kind"] == "frames":
        st["net_out"] = torch.zeros((F, c["height"] * s, c["width"] * s, 3), dtype=torch.float32, device="cuda")
        st["places"], st["n_places"] = rh.identity_places(F)
    if c["kind"] != "plan":
        st["hr"] = torch.zeros((F, c["height"] * s, c["width"] * s, 3), dtype=torch.uint8, device="cuda")
    if c["mode"] in ("needed", "masked"):
        st["sel"] = torch.zeros((mbs, 16 * s, 16 * s, 3), dtype=torch.float32, device="cuda")
    return st


def run(state):
    c, rh = state["case"], state["rh"]
    if c["kind"] == "temporal":
        phi = rh.temporal_phi(state["res"], 12, 1)
        alloc, selected, reuse, n_sel = rh.temporal_select(phi, state["off"], state["total"])
        imp = rh.temporal_spread(state["imp"], selected, reuse)
        return {"phi": phi, "alloc": alloc, "selected": selected, "reuse": reuse, "n_selected": n_sel, "importance": imp}
    if c["kind"] == "frames":
        rh.enhance(state["frames"], out=state["net_out"])
        rh.unpack(state["net_out"], state["places"], state["n_places"], state["frames"], out=state["hr"])
        return {"net": state["net_out"], "places": state["places"]}
    po = state["po"]
    if c["kind"] == "paste":
        hr, _ = rh.unpack(state["net_out"], po.places, po.counts[3:4], state["frames"], out=state["hr"])
        return {"hr": hr}
    mask, lst, n_sel = rh.select_regions(state["imp"], state["segs"])
    rh.pack(state["frames"], state["imp"], mask, lst, n_sel, out=po)
    got = {"mask": mask, "n_selected": n_sel, "bins": po.bins, "boxes": po.boxes, "places": po.places, "counts": po.counts}
    if c["kind"] == "plan":
        return got
    n, n_valid = state["cap"], po.counts[1:2]
    if c["mode"] == "needed":
        rh.enhance_needed(po.bins, po.places, po.counts, n=n, n_valid=n_valid, out=state["net_out"])
    elif c["mode"] == "masked":
        rh.enhance_masked(po.bins, po.boxes, po.counts, n=n, n_valid=n_valid, out=state["net_out"])
    elif c["mode"] == "exact":
        rh.enhance_exact(po.bins, po.boxes, po.counts, n=n, n_valid=n_valid, out=state["net_out"])
    else:
        rh.enhance(po.bins, n=n, n_valid=n_valid, out=state["net_out"])
    # the pasted macroblocks unquantised too, where the program's next stage takes floats; in the needed-region
    # mode they are the only pixels of the network output that are defined
    _, sel = rh.unpack(state["net_out"], po.places, po.counts[3:4], state["frames"], out=state["hr"], want_sel="sel" in state, sel=state.get("sel"))
    if sel is not None:
        got["pasted"] = sel
    if c["mode"] != "needed":
        got["net"] = state["net_out"]
    if c["precision"] == "fp32":
        # 8-bit results are compared where rounding leaves them alone: a bf16 net's own error moves one pasted
        # byte in ten by a level, so there the values before quantisation stand for them (and kind `paste` for the rest)
        got["hr"] = state["hr"]
    return got


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without

def packed_pixels(c, grow=None):
    """Low-resolution pixels of the packed bins.  A region is about 48 pixels wide (16 when the selected
    macroblocks are isolated) and carries its halo (`grow`: only so much of it); the packer fills three quarters
    of a bin (measured occupancy: 0.375 at halo 10 in 128 x 128 bins, 0.52 at halo 6, 0.147 isolated)."""
    px = c["frames"] * ((c["height"] + 15) // 16) * ((c["width"] + 15) // 16) * 256 * c["frac"]
    b, h = (16 if c["importance"] == "scattered" else 48), (c["halo"] if grow is None else min(grow, c["halo"]))
    return px * ((b + 2 * h) / b) ** 2 / (0.75 if grow is None else 1.0)


def work(case):
    c = case
    F, H, W, s, C = c["frames"], c["height"], c["width"], c["scale"], c["channels"]
    mbs = F * ((H + 15) // 16) * ((W + 15) // 16)
    lr, sel_px = 3 * F * H * W, mbs * 256 * c["frac"]
    if c["kind"] == "temporal":
        return {"bytes": 2.0 * F * H * W + 4 * mbs, "flops": 0.0}
    plan_bytes = 5.0 * mbs + 2 * 3 * packed_pixels(c) + (24 + 16) * mbs * c["frac"]
    paste_bytes = lr * (1 + s * s) + sel_px * s * s * 12
    if c["kind"] == "plan":
        return {"bytes": plan_bytes, "flops": 0.0}
    if c["kind"] == "paste":
        return {"bytes": paste_bytes, "flops": 0.0}
    px = float(F * H * W) if c["kind"] == "frames" else packed_pixels(c)
    body = c["blocks"] - 2 if c["topology"] == "plain" else 2 * c["blocks"] + (c["topology"] == "edsr")
    # the linear end of the network is at least one convolution to the 3 s^2 outputs of a pixel (5 x 5 taps for edsr)
    rest = 2 * 27 * C + 2 * C * 3 * s * s * (25 if c["topology"] == "edsr" else 9)
    body_px = px
    if c["mode"] == "needed":       # layer i of the body is needed within i pixels of a pasted one
        body_px = sum(packed_pixels(c, grow=3 + i) for i in range(body)) / max(1, body)
    net_bytes = px * 3 + px * s * s * 12
    return {"bytes": net_bytes + (0 if c["kind"] == "frames" else plan_bytes) + paste_bytes, "flops": body_px * body * 18 * C * C + px * rest}


def tolerance(case):
    if case["kind"] in ("plan", "paste", "temporal"):
        return "exact"
    if case["precision"] == "fp32":
        # sums of up to 1152 products in another order; a pasted byte moves when its value lies that near a half
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    # The same network with the same bf16 activations and its sums in double instead of single precision
    # differs by 0.8 % (16 blocks, 64 channels) and 0.3 % (8 blocks, 32 channels) of the output's norm, largest
    # element 0.044 and 0.023 of its rms over 10^5 values: a last bit that rounds the other way spreads through
    # all later layers.  Up to 10^8 values are compared, whose extremes lie about twice as far out.
    return {"rel": 0.03, "max": 0.3}
