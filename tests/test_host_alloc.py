"""The C entry points' planning allocates no host memory, so that no exception can leave one (tests/host_alloc_check.cpp). CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2604_06694_amd", "libaudiokv.so")


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(LIB), reason="needs g++ and the built library")
def test_planning_allocates_nothing(tmp_path):
    exe = str(tmp_path / "host_alloc_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-rdynamic", "-I", os.path.join(ROOT, "include"),
                        os.path.join(ROOT, "tests", "host_alloc_check.cpp"), "-o", exe, "-ldl"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe, LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "no entry allocates" in r.stdout, (r.returncode, r.stdout, r.stderr)
