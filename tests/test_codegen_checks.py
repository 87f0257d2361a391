"""The look that the build takes at the assembly of the kernels with resident chunk sums (paper_2409_13313_amd/codegen.py): every
instance passes, and what it is there to find is found in assembly with a mistake put in (CPU only: hipcc cross-compiles)."""
import os
import re
import shutil

import pytest

from paper_2409_13313_amd import build, codegen

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
IN_PLACE = "k_extendedILi12ELi12E"


def test_every_instance(resident_assembly):
    total = dict.fromkeys(("k_resident", "k_cut", "k_extended", "k_per_slice"), 0)
    for k, text in resident_assembly.items():
        for kind, count in codegen.check_resident(text, k).items():
            total[kind] += count
    assert total == {"k_resident": 196, "k_cut": 100, "k_extended": 38, "k_per_slice": 26}


def kernel_lines(text, part):
    """(start, end) of the body of the first kernel whose name holds `part`, and its lines"""
    m = next(m for m in codegen.KERNEL.finditer(text) if part in m.group(1))
    return m.start(4), m.end(4), m.group(4).split("\n")


def mfma_lines(lines):
    return [i for i, line in enumerate(lines) if codegen.MFMA in line]


def planted(text, part, put):
    a, b, lines = kernel_lines(text, part)
    put(lines, mfma_lines(lines))
    return text[:a] + "\n".join(lines) + text[b:]


def operands(line):
    return [x.strip() for x in line.split(";")[0].split(codegen.MFMA)[1].split(",")]


def first(register):
    return re.sub(r"\[(\d+):\d+\]", r"\1", register)


MISTAKES = {
    "a chunk sum is copied in the loop": (IN_PLACE, lambda lines, at: lines.insert(at[5] + 1, f"\tv_mov_b32_e32 v0, {first(operands(lines[at[3]])[0])}")),
    "a chunk sum is read before the wait states": (IN_PLACE, lambda lines, at: lines.insert(at[-1] + 1, f"\tv_mov_b32_e32 v0, {first(operands(lines[at[-1]])[0])}")),
    "no wait states": (IN_PLACE, lambda lines, at: lines.__setitem__(slice(at[-1], len(lines)), [x.replace("s_nop 15", "s_nop 0") for x in lines[at[-1]:]])),
    "a fragment is written right before the instruction that reads it": (IN_PLACE, lambda lines, at: lines.insert(at[7] - 1, f"\tv_mov_b32_e32 {first(operands(lines[at[7]])[1])}, v0")),
    "a move between register files": ("k_resident", lambda lines, at: lines.insert(at[4], "\tv_accvgpr_read_b32 v0, a0")),
    "a spill in the loop": ("k_cut", lambda lines, at: lines.insert(at[4], "\tscratch_load_dword v0, off, off")),
    "a wait of the compiler's": ("k_per_slice", lambda lines, at: lines.insert(at[4] - 1, "\ts_waitcnt vmcnt(0)")),
    "another user of M0": ("k_cut", lambda lines, at: lines.insert(at[0] - 40, "\ts_mov_b32 m0, s0")),
}


@pytest.mark.parametrize("mistake", list(MISTAKES))
def test_a_mistake_is_found(resident_assembly, mistake):
    part, put = MISTAKES[mistake]
    with pytest.raises(codegen.Wrong):
        codegen.check_resident(planted(resident_assembly[12], part, put), 12)


def test_an_operand_written_above_the_branch_back_to_the_loop_is_found():
    loop = ["\tv_mov_b32_e32 v9, v8", ".LBB0_1:", "\tv_mfma_i32_16x16x64_i8 a[0:3], v[4:7], v[12:15], a[0:3]", "\ts_nop 1",
            "\tv_mov_b32_e32 v20, v21", "{}", "\ts_cbranch_scc1 .LBB0_1"]
    codegen.check_operands([x.format("\tv_mov_b32_e32 v3, v8") for x in loop], ())
    with pytest.raises(codegen.Wrong):
        codegen.check_operands([x.format("\tv_mov_b32_e32 v5, v8") for x in loop], ())


def test_the_build_makes_no_library_of_wrong_code(monkeypatch, tmp_path):
    class Refuses:
        @staticmethod
        def check_resident(text, k):
            raise codegen.Wrong("planted")
    monkeypatch.setattr(build, "_codegen", lambda: Refuses)
    monkeypatch.setattr(build, "SOURCES", [])
    monkeypatch.setattr(build, "RESIDENT_KS", [3])
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    before = {f: os.path.getmtime(os.path.join(build.CSRC, f)) for f in os.listdir(build.CSRC)}
    with pytest.raises(codegen.Wrong):
        build.build()
    assert not os.path.exists(build.LIB)
    assert before == {f: os.path.getmtime(os.path.join(build.CSRC, f)) for f in os.listdir(build.CSRC)}
