"""Host check of the lane-pair transforms that the plane kernels run, with the kernels' own
exchange (one lane held negated, a signed multiply-add of the other lane's values); and
the kernels hold no other transform."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2104_04547_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_lane_transforms_match_dft(tmp_path):
    exe = str(tmp_path / "fft_lanes_test")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-fsanitize=address,undefined",
                    "-I", CSRC, os.path.join(ROOT, "tests", "csrc", "fft_lanes_test.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr


def test_the_plane_kernels_run_the_tested_transforms():
    src = open(os.path.join(CSRC, "cf_fftconv.hip")).read()
    assert len(re.findall(r"\bfft32_lanes_di[tf]<", src)) >= 10
    assert not re.search(r"void \w*(fft16|fft32|twiddle)\w*\(", src)     # none of its own
