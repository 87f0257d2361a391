"""The look that the build takes at the assembly of k_held (paper_2409_13313_amd/codegen.py): every instance is seen, and a mistake put into one, or
a build without one, is found (CPU only: hipcc cross-compiles)."""
import shutil

import pytest

from paper_2409_13313_amd import codegen
from test_codegen_checks import first, operands, planted

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def test_every_instance_is_looked_at(resident_assembly):
    seen = {k: codegen.check_kernels(text, k)["k_held"] for k, text in resident_assembly.items()}
    assert sum(seen.values()) == 20 and all((seen[k] > 0) == (k in codegen.HELD_KS) for k in seen), seen


MISTAKES = {
    "a chunk sum is copied in the loop": lambda lines, at: lines.insert(at[5] + 1, f"\tv_mov_b32_e32 v0, {first(operands(lines[at[3]])[0])}"),
    "no wait states": lambda lines, at: lines.__setitem__(slice(at[-1], len(lines)), [x.replace("s_nop 15", "s_nop 0") for x in lines[at[-1]:]]),
    "a fragment is written right before the instruction that reads it": lambda lines, at: lines.insert(at[7] - 1, f"\tv_mov_b32_e32 {first(operands(lines[at[7]])[1])}, v0"),
    "another user of M0": lambda lines, at: lines.insert(at[0] - 40, "\ts_mov_b32 m0, s0"),
    "lanes stay off": lambda lines, at: lines.remove(next(x for x in lines if x.strip() == "s_mov_b64 exec, -1")),
}


@pytest.mark.parametrize("mistake", list(MISTAKES))
def test_a_mistake_is_found(resident_assembly, mistake):
    with pytest.raises(codegen.Wrong):
        codegen.check_resident(planted(resident_assembly[12], "k_heldILi12E", MISTAKES[mistake]), 12)


def test_a_build_without_one_is_found(resident_assembly):
    with pytest.raises(codegen.Wrong):
        codegen.check_resident(resident_assembly[12].replace("6k_held", "6k_hold"), 12)
