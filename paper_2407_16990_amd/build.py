"""Build librh.so (the HIP library) in-tree with hipcc for gfx950.

Every source is compiled to an object of its own (in parallel, objects kept under _build/ and
reused while the source, the headers and the flags are unchanged), then linked."""
from __future__ import annotations

import hashlib
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(HERE, "..", "include")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "librh.so")
STAMP = LIB + ".sources"      # digest of the sources the library was built from
SOURCES = ["rh_api.hip", "select.hip", "plan.hip", "pack.hip", "unpack.hip", "conv_fp32.hip", "conv_mfma.hip",
           "conv_mfma_duo.hip", "conv_body.hip", "conv_block32.hip", "conv_block64.hip", "conv_tail.hip", "conv_head.hip", "conv_fold.hip", "conv_mask.hip", "temporal.hip", "noalloc.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=off"]


def _digest(paths, extra: str = "") -> str:
    h = hashlib.sha256(extra.encode())
    for p in paths:
        h.update(os.path.basename(p).encode())
        with open(p, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def _headers():
    return sorted(os.path.join(d, n) for d in (CSRC, INCLUDE) for n in os.listdir(d) if n.endswith(".h"))


def source_digest() -> str:
    """SHA-256 over the names and contents of every file the library is compiled from."""
    return _digest([os.path.join(CSRC, s) for s in SOURCES] + _headers(), " ".join(FLAGS))


SETTLED = 20       # wait states from a matrix product to a vector instruction that reads its sums, more than any product needs


def named_registers(asm: str, first: int) -> int:
    """What conv_block64.hip needs of the compiler and cannot tell it, in the assembly that the compiler made: between the kernel's asm statements it keeps
    nothing in the registers from `first` on, which those statements name themselves, and nothing in scratch memory; no product follows at once on a
    move of what it reads; and on no way through the code are sums read (rounded) before they are settled.  ValueError if not; else the number of kernels."""
    span = lambda t: set(range(int(t[0]), int(t[-1]) + 1))
    inside, written = False, []                              # written: registers that the last vector instructions wrote
    code, labels, kernels = [], {}, 0                        # of the kernel: (instruction, names a register of the kernel's own)
    for line in asm.splitlines():
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
        text = line.split(";")[0].strip()
        if text.startswith(".amdhsa_kernel"):
            _settled(code, labels)
            code, labels, kernels = [], {}, kernels + 1
        if re.match(r"[.\w$]+:$", text):
            labels[text[:-1]] = len(code)
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        named = any(int(m[1] or m[2]) >= first for m in re.finditer(r"\bv(\d+)\b|\bv\[\d+:(\d+)\]", text))
        if named and not inside:
            raise ValueError(f"a register that the kernel names itself is used by the compiler: {text}")
        if text.startswith("scratch_"):
            raise ValueError(f"scratch memory is used: {text}")
        if text.startswith("v_mfma") and any(span(m) & w for m in re.findall(r"v\[(\d+):(\d+)\]", text)[1:3] for w in written[-2:]):
            raise ValueError(f"a product follows at once on a move of what it reads: {text}")
        m = re.match(r"v_(?!mfma|cmp)\w+ v\[?(\d+)(?::(\d+))?", text)
        written.append(span([g for g in m.groups() if g]) if m else set())
        code.append((text, named))
    return kernels


def _settled(code, labels):
    """The fewest wait states from a product to each instruction, over all ways through the code: SETTLED or more at one that reads sums."""
    states, todo = [SETTLED] * len(code), [i + 1 for i, c in enumerate(code[:-1]) if c[0].startswith("v_mfma")]
    for i in todo:
        states[i] = 0
    while todo:
        i = todo.pop()
        op, *arg = code[i][0].split()
        if op in ("s_endpgm", "s_setpc_b64") or op.startswith("v_mfma"):
            continue                                         # what follows a product has its 0 already
        after = states[i] + (int(arg[0]) + 1 if op == "s_nop" else 1)
        for k in ([labels[arg[0]]] if op.startswith(("s_branch", "s_cbranch")) else []) + ([i + 1] if op != "s_branch" else []):
            if k < len(code) and after < states[k]:
                states[k] = after
                todo.append(k)
    for (text, named), n in zip(code, states):
        if named and text.startswith("v_cvt_pk") and n < SETTLED:
            raise ValueError(f"sums are read {n} wait states behind a product: {text}")


def _checked(hipcc: str, src: str) -> None:
    """The checks of a source whose kernels name registers themselves, on what this compiler makes of it."""
    first = re.search(r"#define B64_X (\d+)", open(os.path.join(CSRC, src)).read())
    if not first:
        return
    r = subprocess.run([hipcc] + FLAGS + ["-I" + INCLUDE, "-I" + CSRC, "-S", "--cuda-device-only", os.path.join(CSRC, src), "-o", "-"], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}{r.stderr}")
    try:
        named_registers(r.stdout, int(first[1]))
    except ValueError as e:
        raise RuntimeError(f"{src}: this compiler's code does not keep what the source relies on: {e}")


def _compile(hipcc: str, src: str, force: bool):
    obj = os.path.join(OBJ, src.replace(".hip", ".o"))
    tag = _digest([os.path.join(CSRC, src)] + _headers(), " ".join(FLAGS))
    if not force and os.path.exists(obj) and os.path.exists(obj + ".tag") and open(obj + ".tag").read() == tag:
        return obj, ""
    cmd = [hipcc] + FLAGS + ["-I" + INCLUDE, "-I" + CSRC, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}{r.stderr}")
    _checked(hipcc, src)
    with open(obj + ".tag", "w") as f:
        f.write(tag)
    return obj, r.stdout + r.stderr


def build(verbose: bool = False, force: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    jobs = min(8, int(os.environ.get("MAX_JOBS", "8")), len(SOURCES))
    with ThreadPoolExecutor(jobs) as ex:
        res = list(ex.map(lambda s: _compile(hipcc, s, force), SOURCES))
    if verbose:
        sys.stderr.write("".join(log for _, log in res))
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + [o for o, _ in res],
                       capture_output=True, text=True)
    if verbose or r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed linking librh.so")
    with open(STAMP, "w") as f:
        f.write(source_digest() + "\n")
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv, force="--force" in sys.argv))
