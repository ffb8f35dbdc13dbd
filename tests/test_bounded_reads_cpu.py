"""Reads that may pass the end of a caller's array are range-checked by the hardware: in the
built top-k kernel every buffer load has its whole offset in the vector operand, since the
scalar offset of a raw buffer load is not part of the range check."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2104_04547_amd", "libcf.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.mark.skipif(not os.path.exists(OBJDUMP) or not os.path.exists(LIB), reason="built library or llvm-objdump absent")
def test_top_k_reads_have_no_scalar_offset(tmp_path):
    lib = shutil.copy(LIB, tmp_path)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=tmp_path)
    loads = {}
    for obj in glob.glob(str(tmp_path / "*gfx950*")):
        syms = subprocess.run([OBJDUMP, "--syms", obj], check=True, capture_output=True, text=True).stdout
        names = [s.split()[-1] for s in syms.splitlines() if "k_topk_small" in s and not s.endswith(".kd")]
        if not names:
            continue
        text = subprocess.run([OBJDUMP, "--disassemble", "--disassemble-symbols=" + ",".join(names), obj], check=True,
                              capture_output=True, text=True).stdout
        for line in text.splitlines():
            m = re.match(r"\s*buffer_load_\w+\s+([^/]*)", line)
            if m:
                ops = [o.strip() for o in m.group(1).split(",")]
                loads[line.strip()] = ops[3].split()[0]      # vdata, vaddr, srsrc, soffset
    assert len(loads) >= 3, "no buffer loads found in k_topk_small"
    bad = [line for line, soffset in loads.items() if soffset != "0"]
    assert not bad, bad[:3]


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="hipcc absent")
@pytest.mark.parametrize("name,steps", [("kConvPadSteps", 15), ("kConvPadTaps", 3)])
def test_conv_weight_prefetch_stays_within_the_padding(tmp_path, name, steps):
    """The deepest prefetch equals the padding of the packed weights: with one step less
    the kernels do not compile."""
    shutil.copytree(os.path.join(ROOT, "include"), tmp_path / "include")
    csrc = shutil.copytree(os.path.join(ROOT, "paper_2104_04547_amd", "csrc"), tmp_path / "a" / "csrc")
    header = os.path.join(csrc, "cf_internal.h")
    text, n = re.subn(rf"constexpr int {name} = \d+;", f"constexpr int {name} = {steps};", open(header).read())
    assert n == 1
    with open(header, "w") as f:
        f.write(text)
    r = subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "--cuda-device-only",
                        "-I", str(tmp_path / "include"), os.path.join(csrc, "cf_conv.hip")], capture_output=True, text=True)
    assert r.returncode != 0 and "prefetch past the weight padding" in r.stderr, r.stderr[-2000:]
