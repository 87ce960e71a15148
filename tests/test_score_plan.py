"""The key ranges that score plans for items of different lengths (tests/score_plan_check.cpp against the built library). CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2604_06694_amd")
LIB = os.path.join(PKG, "libaudiokv.so")


@pytest.mark.skipif(shutil.which("hipcc") is None or not os.path.exists(LIB), reason="needs hipcc and the built library")
def test_division_of_ragged_items(tmp_path):
    exe = str(tmp_path / "score_plan_check")
    r = subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++20", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(PKG, "csrc"), os.path.join(ROOT, "tests", "score_plan_check.cpp"), "-x", "none", LIB,
                        f"-Wl,-rpath,{PKG}", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "the ranges are as planned" in r.stdout, (r.returncode, r.stdout[-2000:], r.stderr)
