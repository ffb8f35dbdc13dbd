"""Host check of the radix select's digit choice, built with g++ from the kernels' own
header: the threads of a workgroup write the select state in any order and the result must
not depend on it; and the kernel reads that state before the barriers of the pass."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2104_04547_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_digit_choice_does_not_depend_on_the_threads_order(tmp_path):
    exe = str(tmp_path / "topk_pick_test")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-fsanitize=address,undefined", "-I", CSRC,
                    os.path.join(ROOT, "tests", "csrc", "topk_pick_test.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr


def test_the_digit_kernel_reads_the_state_before_its_barriers():
    src = open(os.path.join(CSRC, "cf_select.hip")).read()
    body = re.search(r"void k_topk_digit\(.*?\n}\n", src, re.S).group(0)
    last = body.rindex("__syncthreads()")
    # past the last barrier the state is only written (by topk_pick's one thread)
    assert not re.search(r"state\[[0-2]\]", body[last:])
    assert all(f"state[{i}]" in body[:last] for i in range(3))
