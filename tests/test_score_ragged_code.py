"""The score kernels for items of different lengths and those that keep a tile on its way across barriers: what
tests/test_kernel_code.py and tests/test_score_ring.py hold the others to, and the order of the latter. CPU only."""
import os
import re
import shutil
import subprocess

import pytest

from test_kernel_code import LLVM, assembly, code_objects, named, pytestmark as needs_library, resources  # noqa: F401

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


def successors(i, what, target, flags):
    """What may follow an instruction, with the truth values in scalar registers as far as they are known: (index, flags)."""
    what = re.sub(r"\s+", " ", what)
    known = dict(flags)
    mask = re.match(r"s_(andn2|and)_b64 vcc, exec, (s\[\d+:\d+\])$", what)
    value = known.get(mask.group(2)) if mask else None
    written = re.match(r"[sv]_\S+ (?:s(\d+)\b|s\[(\d+):(\d+)\]|(vcc))", what)
    if written:
        lo, hi = int(written.group(1) or written.group(2) or -1), int(written.group(1) or written.group(3) or -1)
        for reg in list(known):
            span = re.match(r"s\[(\d+):(\d+)\]", reg)
            if reg == written.group(4) or (span and lo >= 0 and int(span.group(1)) <= hi and lo <= int(span.group(2))):
                del known[reg]
    const = re.match(r"s_mov_b64 (s\[\d+:\d+\]), (0|-1)$", what)
    if const:
        known[const.group(1)] = const.group(2) == "-1"
    elif value is not None:
        known["vcc"] = value == (mask.group(1) == "and")
    flags = tuple(sorted(known.items()))
    if what.startswith("s_endpgm"):
        return []
    if target is None:
        return [(i + 1, flags)]
    taken = {"s_branch": True, "s_cbranch_execnz": True, "s_cbranch_execz": False}.get(what.split()[0])     # (a wave has lanes)
    if "vcc" in known and what.startswith("s_cbranch_vcc"):
        taken = known["vcc"] == what.startswith("s_cbranch_vccnz")
    return [(target, flags)] * (taken is not False) + [(i + 1, flags)] * (taken is not True)


@needs_library
def test_no_tile_passes_a_barrier_without_a_wait(code_objects):  # noqa: F811
    """Tiles in flight across barriers: on every path through the loader, a wait stands between the last load and the barrier after it
    and between two barriers, and one that leaves sixteen loads on their way follows the sixteen of a newest tile."""
    seen = 0
    for f in code_objects:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "-C", f], check=True, capture_output=True, text=True).stdout
        for block in re.split(r"\n\n(?=[0-9a-f]+ <)", text):
            name = re.search(r"<(.+)>:\n", block)
            if not name or not re.search(r"score_(ragged|ahead)_kernel<256, 1, [478], ", name.group(1)):
                continue
            seen += 1
            rows = [re.match(r"\s*(\S.*?)\s*// ([0-9A-F]+):", line) for line in block.splitlines()[1:]]
            rows = [(m.group(1), int(m.group(2), 16)) for m in rows if m]
            index = {at: i for i, (_, at) in enumerate(rows)}
            first = next(i for i, (what, _) in enumerate(rows) if what.startswith("global_load_lds"))
            # (instruction; loads since the last barrier; whether they were waited for; the least that a wait for all but a tile's follows;
            # known flags. That it is 48 before the first barrier depends on comparisons with the number of tiles, which are not followed.)
            todo, met, passed = [(first, 0, False, 32, ())], set(), {"0": 0, "16": 0}
            while todo:
                state = todo.pop()
                if state in met:
                    continue
                met.add(state)
                i, loads, waited, newest, flags = state
                what, at = rows[i]
                wait = re.match(r"s_waitcnt .*?vmcnt\((\d+)\)", what)
                if what.startswith("global_load_lds"):
                    loads, waited = loads + 1, False
                    assert loads <= 48, (name.group(1), i, loads)
                elif wait:
                    assert wait.group(1) == "0" or (wait.group(1) == "16" and loads >= newest), (name.group(1), i, what, loads)
                    passed[wait.group(1)] += 1
                    waited = True
                elif what.startswith("s_barrier"):
                    assert waited, (name.group(1), i, loads)
                    loads, waited, newest = 0, False, 16
                jump = re.match(r"s_c?branch\S* (\d+)$", re.sub(r"\s+", " ", what))
                target = index[at + 4 + 4 * ((int(jump.group(1)) ^ 0x8000) - 0x8000)] if jump else None
                todo += [(n, loads, waited, newest, known) for n, known in successors(i, what, target, flags)]
            assert passed["0"] and passed["16"], (name.group(1), passed)
    assert seen == 12, seen
