"""The roots of unity of the smoothing's transforms are evaluated in float64 and rounded to float32 once: csrc/fft_regs.h
compiled for the host and compared with long double (tests/fft_roots_check.cpp). CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_roots_are_rounded_once(tmp_path):
    exe = str(tmp_path / "fft_roots_check")
    r = subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++20", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                        os.path.join(ROOT, "paper_2604_06694_amd", "csrc"), os.path.join(ROOT, "tests", "fft_roots_check.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "all bounds hold" in r.stdout, r.stdout + r.stderr
