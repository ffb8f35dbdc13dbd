"""Host check of the launch sizes of work-item loops, built with g++ from the library's own
header; and the launches over (pose, block of atoms) items take their size from there."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2104_04547_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_item_launches_stay_below_the_thread_limit(tmp_path):
    exe = str(tmp_path / "launch_test")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined", "-I", CSRC,
                    os.path.join(ROOT, "tests", "csrc", "launch_test.cpp"), "-o", exe], check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr


@pytest.mark.parametrize("source,kernels", [("cf_splat.hip", ["k_splat_bin"]), ("cf_graph.hip", ["k_graph_count", "k_graph_fill"]),
                                            ("cf_select.hip", ["k_segmax"])])
def test_item_kernels_are_launched_with_them(source, kernels):
    """A whole batch of any size goes to these kernels in one launch."""
    src = open(os.path.join(CSRC, source)).read()
    sized = set(re.findall(r"(\w+)(?: =|\()\s*item_groups\(", src))        # variables that hold such a size
    for k in kernels:
        grids = re.findall(rf"hipLaunchKernelGGL\(\(?{k}\b[^,]*,\s*(.*?), dim3\(k", src, re.S)
        assert grids
        for g in grids:
            assert "item_groups(" in g or any(re.search(rf"\b{v}\b", g) for v in sized), (k, g)
