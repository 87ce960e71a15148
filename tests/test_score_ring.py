"""The hand-over of key tiles inside the score kernels: csrc/score_ring.h compiled for the host (tests/score_ring_check.cpp), and
the waits that the kernels of the built library have in front of the loader wave's barriers. CPU only."""
import os
import re
import shutil
import subprocess

import pytest

from test_kernel_code import assembly, code_objects, named, pytestmark as needs_library  # noqa: F401

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_tiles_have_landed_when_they_are_read(tmp_path):
    exe = str(tmp_path / "score_ring_check")
    r = subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++20", "-O1", "-I",
                        os.path.join(ROOT, "paper_2604_06694_amd", "csrc"), os.path.join(ROOT, "tests", "score_ring_check.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "the ring holds" in r.stdout, r.stdout + r.stderr


@needs_library
def test_loader_waits_for_what_it_requested(assembly):  # noqa: F811
    for name, lines in named(assembly, "score_kernel<").items():
        loads = [i for i, line in enumerate(lines) if line.startswith("global_load_lds")]
        assert loads, name
        # the barriers between the loader's first and last request, and the one behind them
        barriers = [i for i, line in enumerate(lines) if line.startswith("s_barrier") and i > loads[0]]
        barriers = [i for i in barriers if i < loads[-1]] + [i for i in barriers if i > loads[-1]][:1]
        assert len(barriers) >= 2, name
        for i in barriers:
            waits = [line for line in lines[max(0, i - 6):i] if re.match(r"s_waitcnt .*vmcnt\(0\)", line)]
            assert waits, (name, lines[max(0, i - 6):i + 1])
