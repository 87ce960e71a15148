"""The score kernels for items of different lengths and those that keep a tile on its way across barriers: what
tests/test_kernel_code.py and tests/test_score_ring.py hold the others to, and the order of the latter. CPU only."""
import os
import re
import shutil
import subprocess

import pytest

from test_kernel_code import assembly, code_objects, named, pytestmark as needs_library, resources  # noqa: F401

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_tiles_have_landed_when_they_are_read(tmp_path):
    exe = str(tmp_path / "score_ring_ahead_check")
    r = subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++20", "-O1", "-I",
                        os.path.join(ROOT, "paper_2604_06694_amd", "csrc"), os.path.join(ROOT, "tests", "score_ring_ahead_check.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "the ring holds" in r.stdout, r.stdout + r.stderr


@needs_library
def test_no_spills_and_no_lost_workgroups(resources):  # noqa: F811
    for name, (vgprs, spills, _) in {**named(resources, "score_ragged_kernel<"), **named(resources, "score_ahead_kernel<")}.items():
        assert spills == 0, (name, spills)
        if re.search(r"<256, 1, [124], true>", name):
            assert vgprs <= 168, (name, vgprs)
        if re.search(r"<(64|128), 1, \d, ", name):
            assert vgprs <= 128, (name, vgprs)


@needs_library
def test_loader_waits_for_what_is_read_next(assembly):  # noqa: F811
    """All that was requested, or all but the sixteen loads of the newest tile at d = 256 with four compute waves and more."""
    for name, lines in {**named(assembly, "score_ragged_kernel<"), **named(assembly, "score_ahead_kernel<")}.items():
        ahead = re.search(r"<256, 1, [478], ", name)
        loads = [i for i, line in enumerate(lines) if line.startswith("global_load_lds")]
        barriers = [i for i, line in enumerate(lines) if line.startswith("s_barrier") and i > loads[0]]
        barriers = [i for i in barriers if i < loads[-1]] + [i for i in barriers if i > loads[-1]][:1]
        assert len(barriers) >= 2, name
        if not ahead:
            for i in barriers:
                assert any(re.match(r"s_waitcnt .*vmcnt\(0\)", line) for line in lines[max(0, i - 6):i]), (name, lines[max(0, i - 6):i + 1])
        else:
            # both waits, and no other one between the loader's loads
            waits = {m.group(1) for line in lines[loads[0]:barriers[-1]] for m in [re.match(r"s_waitcnt .*?vmcnt\((\d+)\)", line)] if m}
            assert waits == {"0", "16"}, (name, waits)
