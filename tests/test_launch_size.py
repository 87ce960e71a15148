"""Sizes of launches that take other work along (tests/launch_size_check.cpp): csrc/conv_filter.h compiled for the host. CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_riders_fit_the_launch(tmp_path):
    exe = str(tmp_path / "launch_size_check")
    r = subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++20", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_2604_06694_amd", "csrc"), os.path.join(ROOT, "tests", "launch_size_check.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "launches hold" in r.stdout, (r.returncode, r.stdout[-2000:], r.stderr)
