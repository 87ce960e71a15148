"""The score kernels for items of different lengths, as compiled: what tests/test_kernel_code.py and tests/test_score_ring.py hold the
others to. CPU only."""
import re

from test_kernel_code import assembly, code_objects, named, pytestmark, resources  # noqa: F401


def test_no_spills_and_no_lost_workgroups(resources):  # noqa: F811
    for name, (vgprs, spills, _) in named(resources, "score_ragged_kernel<").items():
        assert spills == 0, (name, spills)
        if re.search(r"<256, 1, [124], true>", name):
            assert vgprs <= 168, (name, vgprs)
        if re.search(r"<(64|128), 1, \d, ", name):
            assert vgprs <= 128, (name, vgprs)


def test_loader_waits_for_what_it_requested(assembly):  # noqa: F811
    for name, lines in named(assembly, "score_ragged_kernel<").items():
        loads = [i for i, line in enumerate(lines) if line.startswith("global_load_lds")]
        barriers = [i for i, line in enumerate(lines) if line.startswith("s_barrier") and i > loads[0]]
        barriers = [i for i in barriers if i < loads[-1]] + [i for i in barriers if i > loads[-1]][:1]
        assert len(barriers) >= 2, name
        for i in barriers:
            assert any(re.match(r"s_waitcnt .*vmcnt\(0\)", line) for line in lines[max(0, i - 6):i]), (name, lines[max(0, i - 6):i + 1])
