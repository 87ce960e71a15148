"""The launches that smooth and select in one workgroup: the waves that the transform does not need pass as many barriers as it has,
read from the built kernels, where a count that is off by one would be a race or a hang. CPU only."""
import re
import subprocess

import pytest

from test_kernel_code import LLVM, code_objects, named, pytestmark, resources  # noqa: F401

FUSED = {f"smooth_select_kernel<{n}>" for n in range(9, 14)} | {f"conv_select_kernel<{n}, {s}>" for n in (10, 11, 12) for s in ("true", "false")}


@pytest.fixture(scope="module")
def listings(code_objects):  # noqa: F811
    """Fused kernel -> its instructions and, for branches, the index of the target: (text, target)."""
    out = {}
    for f in code_objects:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "-C", f], check=True, capture_output=True, text=True).stdout
        for block in re.split(r"\n\n(?=[0-9a-f]+ <)", text):
            name = re.search(r"<(?:.*::)?(\w+_select_kernel<[^>]*>)\(.*>:\n", block)
            if not name:
                continue
            rows = [re.match(r"\s*(\S.*?)\s*// ([0-9A-F]+):", line) for line in block.splitlines()[1:]]
            rows = [(m.group(1), int(m.group(2), 16)) for m in rows if m]
            index = {at: i for i, (_, at) in enumerate(rows)}
            code = []
            for what, at in rows:
                jump = re.match(r"s_c?branch\S* (\d+)$", re.sub(r"\s+", " ", what))
                # (a signed number of words past the branch itself)
                code.append((what, index[at + 4 + 4 * ((int(jump.group(1)) ^ 0x8000) - 0x8000)] if jump else None))
            out[name.group(1)] = code
    return out


def test_all_fused_kernels_are_there(listings):
    assert set(listings) == FUSED


@pytest.mark.parametrize("name", sorted(FUSED))
def test_idle_waves_pass_every_barrier(listings, name):
    code = listings[name]
    barriers = [i for i, (what, _) in enumerate(code) if what.startswith("s_barrier")]
    # the idle waves: a loop of one barrier, counted down from a constant
    first = barriers[0]
    back = next(i for i in range(first, first + 4) if code[i][1] is not None and code[i][1] <= first)
    start = code[back][1]
    assert [i for i in barriers if start <= i <= back] == [first]
    counter = next(m for i in range(start, back) for m in [re.match(r"s_add_i32 (s\d+), \1, -1$", code[i][0])] if m).group(1)
    assert any(re.match(rf"s_cmp_lg_u32 {counter}, 0$", code[i][0]) for i in range(start, back))
    count = next(m for i in range(start - 1, start - 5, -1) for m in [re.match(rf"s_movk?_[bi]32 {counter}, (\w+)$", code[i][0])] if m).group(1)
    # and then past the transform, on every path through which the others pass as many (not the one of waves without lanes)
    skip = next(i for i in range(back + 1, back + 12) if code[i][1] is not None and code[i][1] > i)
    end = code[skip][1]
    passed, todo, at_the_end = set(), [(skip + 1, 0)], set()
    while todo:
        i, n = todo.pop()
        if i == end:
            at_the_end.add(n)
            continue
        if (i, n) in passed:
            continue
        passed.add((i, n))
        what, target = code[i]
        assert skip < i < end and n <= int(count, 0) and not what.startswith(("s_endpgm", "s_setpc")), (name, i, n, what)
        if target is not None and not (target == end and what.startswith("s_cbranch_execz")):
            todo.append((target, n))
        if not what.startswith("s_branch"):
            todo.append((i + 1, n + what.startswith("s_barrier")))
    assert at_the_end == {int(count, 0)}, (name, at_the_end, count)


def test_fused_kernels_do_not_spill(resources):  # noqa: F811
    for name, (vgprs, spills, threads) in {**named(resources, "smooth_select_kernel<"), **named(resources, "conv_select_kernel<")}.items():
        assert spills == 0 and (threads <= 512 or vgprs <= 128), (name, vgprs, spills)
