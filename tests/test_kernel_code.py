"""What the compiler made of the kernels, read from this package's own library: properties that results do not show, since a
violation is an access that only happens to be harmless, or a lost workgroup per CU. CPU only."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2604_06694_amd", "libaudiokv.so")
LLVM = "/opt/rocm/llvm/bin"

pytestmark = pytest.mark.skipif(not os.path.exists(LIB) or not os.path.exists(os.path.join(LLVM, "llvm-objdump")),
                                reason="needs the built library and llvm-objdump")


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    d = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, d / "lib.so")
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    found = sorted(str(d / f) for f in os.listdir(d) if f.endswith("gfx950"))
    assert found
    return found


@pytest.fixture(scope="module")
def assembly(code_objects):
    """Kernel or function -> its instructions."""
    out = {}
    for f in code_objects:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "-C", "--no-show-raw-insn", f], check=True, capture_output=True, text=True).stdout
        for block in re.split(r"\n\n(?=[0-9a-f]+ <)", text):
            name = re.search(r"<(.+)>:\n", block)
            if name:
                out[name.group(1)] = [line.split("//")[0].strip() for line in block.splitlines()[1:]]
    return out


def named(table, part):
    some = {k: v for k, v in table.items() if part in k}
    assert some, part
    return some


def test_buffer_offsets_are_range_checked(assembly):
    """Buffers are sized so that what lies past a head's end reads as zero or is not stored. The scalar offset of a buffer
    instruction is no part of that check, so none may be used: the offsets are all in the vector operand (or constant)."""
    seen = 0
    for name, lines in assembly.items():
        for line in lines:
            if re.match(r"buffer_(load|store)_", line):
                seen += 1
                operands = line.split("s[", 1)[1]                  # resource, scalar offset, modifiers
                assert re.match(r"\d+:\d+\], 0( |$)", operands), (name, line)
    assert seen > 0


@pytest.fixture(scope="module")
def resources(code_objects):
    """Kernel -> (vector registers, spilled vector registers, threads of its largest workgroup)."""
    out = {}
    for f in code_objects:
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", f], check=True, capture_output=True, text=True).stdout
        for kernel in re.split(r"\n  - (?=\.)", notes)[1:]:
            def value(key):
                return re.search(rf"^\s*{re.escape(key)}:\s+(\S+)", kernel, re.M).group(1)
            name = subprocess.run(["c++filt", value(".name").strip("'")], check=True, capture_output=True, text=True).stdout.strip()
            out[name] = int(value(".vgpr_count")), int(value(".vgpr_spill_count")), int(value(".max_flat_workgroup_size"))
    return out


def test_score_kernels_keep_their_registers(resources):
    """No spills, and at head_dim 256 three waves per SIMD (512 registers) where that decides how many workgroups share a CU."""
    for name, (vgprs, spills, _) in named(resources, "score_kernel<").items():
        assert spills == 0, (name, spills)
        if re.search(r"<256, 1, [124], true>", name):
            assert vgprs <= 168, (name, vgprs)


def test_smoothing_kernels_keep_their_registers(resources):
    """Power-of-two heads up to 16384 samples: no spills, and never more than 128 registers, with which the workgroups of up to 512
    threads fill a CU twice. (32768 samples, sixteen points per thread, spill.)"""
    for name, (vgprs, spills, _) in named(resources, "smooth_real_kernel<").items():
        if not re.search(r"smooth_real_kernel<14, ", name):
            assert spills == 0 and vgprs <= 128, (name, vgprs, spills)
