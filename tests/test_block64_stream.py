"""The row streams of k_conv_mfma_block64 (conv_block64.hip) on the CPU: which input row lies in which place, which row of the tensor between a product reads,
when an output row is finished, rounded and stored, and what columns beside a strip or an image hold - with one channel and whole
numbers, so that every output must be exact.  And of the compiled kernel: that the compiler keeps nothing in the registers that the kernel
names itself, which build() checks too."""
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2407_16990_amd import build

RING = 7


def conv(x, w):
    p = np.pad(x, 1)
    return sum(w[i, j] * p[i:i + x.shape[0], j:j + x.shape[1]] for i in range(3) for j in range(3))


def strips_of(W):
    """rh_block64_strips: strips, columns of one, tiles of conv1 and of conv2"""
    best = None
    for n in range(1, (W + 47) // 48 + 1):
        w = -(-W // n)
        nt1, nt2 = -(-(w + (n > 1) + (n > 2)) // 16), -(-w // 16)
        if 4 <= nt1 <= 8 and (n - 1) * w < W and (best is None or n * (nt1 + nt2) < best[0]):
            best = (n * (nt1 + nt2), n, w, nt1, nt2)
    return best and best[1:]


class Stream:
    def __init__(self, pos, end, H, strips):
        self.pos, self.end, self.H, self.strips = pos, end, H, strips
        self.c = None
        self.piece()

    def piece(self):
        if self.pos >= self.end:
            self.c = None
            return
        col = self.pos // self.H
        y0 = self.pos - col * self.H
        y1 = min(self.H, y0 + self.end - self.pos)
        self.c = dict(n=col // self.strips, s=col % self.strips, y0=y0, y1=y1, r=max(y0 - 2, -1))
        self.pos += y1 - y0

    def next(self):
        if self.c is None:
            return
        self.c = dict(self.c, r=self.c["r"] + 1)
        if self.c["r"] > min(self.c["y1"], self.H - 1) + 1:
            self.piece()


class Sums:
    """of the row that is finished next (Y) and of the newest (Z); a row of input moves them on"""

    def __init__(self, n):
        self.Y, self.Z = np.full(n, np.nan), np.full(n, np.nan)

    def take(self, w, row):
        j = np.arange(len(self.Y))
        part = lambda ky: 0 if row is None else sum(w[ky, kx] * row[j + kx] for kx in range(3))
        X, self.Y, self.Z = self.Y + part(2), self.Z + part(1), np.zeros(len(j)) + part(0)
        return X


def run(x, w1, w2, G):
    N, H, W = x.shape
    strips, wo, nt, nt2 = strips_of(W)
    px = 16 * nt + 8
    out = np.full(x.shape, np.nan)
    total = N * strips * H
    for wg in range(G):
        share, more = total // G, total % G
        pos = wg * share + min(wg, more)
        end = pos + share + (wg < more)
        if pos >= end:
            continue
        ring, mid = np.full((RING, px), np.nan), np.full((2, px), np.nan)
        left = lambda s: 1 if s > 0 else 0

        def copy(c, slot):
            if c is None or not 0 <= c["r"] < H:
                return
            gx = c["s"] * wo - left(c["s"]) - 1 + np.arange(px)
            ring[slot] = np.where((gx >= 0) & (gx < W), x[c["n"], c["r"], np.clip(gx, 0, W - 1)], 0)

        st = Stream(pos, end, H, strips)
        rows = []
        while st.c is not None:
            rows.append(st.c)
            st.next()
        at = lambda t: rows[t] if 0 <= t < len(rows) else None
        inside = lambda c: c is not None and 0 <= c["r"] < H
        copy(at(0), 0)
        S1, S2 = Sums(16 * nt), Sums(16 * nt2)
        X = np.full(16 * nt2, np.nan)                        # conv2's sums of the row that it finished last
        done = rounded = last = None
        for t in range(len(rows) + 4):
            before, c, slot, par = at(t - 1), at(t), t % RING, t & 1
            # conv1 stores what conv2 rounded in the last iteration
            if rounded:
                xo = rounded["s"] * wo
                k = np.arange(min(wo, W - xo))
                assert np.isnan(out[rounded["n"], rounded["y"], xo + k]).all()
                out[rounded["n"], rounded["y"], xo + k] = ring[(slot + 2) % RING, k + left(rounded["s"]) + 1]
            # conv2 rounds what it finished in the last iteration, and reads what conv1 left then
            if done:
                ci = np.arange(16 * nt2) + left(done["s"]) + 1
                assert ci.max() < px
                ring[(slot + 3) % RING, ci] += X
            q, rounded, done, what = (before["r"] - 1 if before else 0), done, None, None
            if before and q >= max(before["y0"] - 1, 0):
                what = "products"
                if q > before["y0"]:
                    done = dict(n=before["n"], s=before["s"], y=q - 1)
                if q == H - 1 and before["y1"] == H:
                    last = dict(n=before["n"], s=before["s"], y=q)
            elif last:
                what, done, last = "zeros", last, None
            elif before and q == -1:
                what = "zeros"
            if what:                                         # nothing: the sums stay as they are
                X = S2.take(w2, mid[par ^ 1] if what == "products" else None)
            # conv1
            if c:
                Y = S1.take(w1, ring[slot] if inside(c) else None)
                xs, shift, right = c["s"] * wo - left(c["s"]), 1 - left(c["s"]), W - c["s"] * wo + 1
                j = np.arange(16 * nt)
                mid[par, j + shift] = np.where(xs + j < W, np.maximum(Y, 0), 0)
                if shift:
                    mid[par, 0] = 0
                if 16 * nt + shift <= right < px:
                    mid[par, right] = 0
            copy(at(t + 1), (slot + 1) % RING)               # last: the place must not be read in this iteration
        assert done is None and rounded is None and last is None
    return out


@pytest.mark.parametrize("N,H,W,G", [(1, 1, 50, 3), (2, 2, 64, 5), (3, 9, 128, 8), (2, 37, 96, 16), (1, 23, 130, 7), (2, 16, 160, 5), (1, 14, 333, 9),
                                     (5, 5, 100, 2), (1, 40, 480, 13), (3, 3, 640, 24), (4, 12, 127, 1), (2, 7, 129, 64)])
def test_every_row_once_and_exact(N, H, W, G):
    rng = np.random.default_rng(N * 1000 + W)
    x = rng.integers(-3, 4, (N, H, W)).astype(float)
    w1, w2 = rng.integers(-2, 3, (3, 3)).astype(float), rng.integers(-2, 3, (3, 3)).astype(float)
    got = run(x, w1, w2, G)
    for n in range(N):
        assert np.array_equal(got[n], x[n] + conv(np.maximum(conv(x[n], w1), 0), w2))


def test_strips_cover_every_width():
    for W in range(49, 2000):
        strips, wo, nt, nt2 = strips_of(W)
        assert strips * wo >= W > (strips - 1) * wo and wo + (strips > 1) + (strips > 2) <= 16 * nt <= 128
        assert wo <= 16 * nt2 and nt2 in (nt - 1, nt)


@pytest.fixture(scope="module")
def assembly():
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS + ["-I" + build.INCLUDE, "-I" + build.CSRC, "-S", "--cuda-device-only",
                        os.path.join(build.CSRC, "conv_block64.hip"), "-o", "-"], check=True, capture_output=True, text=True)
    return r.stdout


FIRST = int(re.search(r"#define B64_X (\d+)", open(os.path.join(build.CSRC, "conv_block64.hip")).read())[1])


def test_the_compiler_keeps_out_of_the_named_registers(assembly):
    assert build.named_registers(assembly, FIRST) >= 20


# Each planted in the compiler's code of one kernel: what build() has to refuse
def test_the_check_finds_what_it_is_for(assembly):
    lines = assembly[:assembly.index(".end_amdhsa_kernel")].splitlines()
    code = lambda i: lines[i].split(";")[0].strip()
    assert build.named_registers("\n".join(lines), FIRST) == 1
    cvt = [i for i in range(len(lines)) if code(i).startswith("v_cvt_pk") and int(re.search(r", v(\d+),", code(i))[1]) >= FIRST]
    mfma = next(i for i in range(len(lines)) if code(i).startswith("v_mfma"))
    start = next(i for i in range(mfma, 0, -1) if "#ASMSTART" in lines[i])
    operand = re.findall(r"v\[(\d+):", code(mfma))[1]
    put = lambda at, *what: lines[:at] + list(what) + lines[at:]
    bad = {"registers": put(start, f"\tv_mov_b32_e32 v{FIRST + 7}, v1"), "scratch": put(start, "\tscratch_load_dword v1, off, off"),
           "move": put(start, f"\tv_mov_b32_e32 v{operand}, v1"),
           "product just before conv1's rounding": put(cvt[0], code(mfma), "\ts_nop 15"), "before conv2's": put(cvt[-1], code(mfma), "\ts_nop 3")}
    around = list(lines)
    for at, what in sorted([(cvt[0], ".Lround:"), (mfma + 1, "\ts_cbranch_scc1 .Lround")], reverse=True):
        around.insert(at, what)
    bad["a way around the waits"] = around
    for what, text in bad.items():
        with pytest.raises(ValueError):
            build.named_registers("\n".join(text), FIRST)
            pytest.fail(what)
    build.named_registers("\n".join(put(cvt[0], code(mfma), "\ts_nop 15", "\ts_nop 3")), FIRST)
