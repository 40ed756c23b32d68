"""What the compiler reports of the kernels whose sums fill the registers: nothing of theirs is kept in scratch memory, from where every unit or tile
would load it again."""
import os
import re
import subprocess

import pytest

from paper_2407_16990_amd import build


def resources(source, out):
    """kernel -> {figure of its metadata: value}"""
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + build.FLAGS + ["-I" + build.INCLUDE, "-I" + build.CSRC, "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, source), "-o", str(out)], check=True, capture_output=True)
    found = {}
    for part in out.read_text().split("  - .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", part)[1]
        found[name] = {k: int(re.search(r"\." + k + r":\s+(\d+)", part)[1]) for k in ("private_segment_fixed_size", "vgpr_spill_count")}
    return found


@pytest.mark.parametrize("source,kernel,how_many", [("conv_body.hip", "k_conv_mfma_body", 2), ("conv_fold.hip", "k_conv_fold", 9)])
def test_no_scratch_memory(source, kernel, how_many, tmp_path):
    found = {n: r for n, r in resources(source, tmp_path / "k.s").items() if kernel in n}
    assert len(found) == how_many
    assert not {n: r for n, r in found.items() if any(r.values())}


def test_asm_that_sets_m0_says_so():
    found = 0
    for name in sorted(os.listdir(build.CSRC)):
        text = open(os.path.join(build.CSRC, name)).read()
        for m in re.finditer(r"\basm\s*(?:volatile)?\s*\((.*?)\);", text, re.S):
            if re.search(r'"\s*s_\w+ m0,', m[1]):
                found += 1
                assert re.search(r'"m0"[^:]*$', m[1]), (name, m[1])
    assert found >= 4
