"""Code-generation checks of k_extended (CPU only: hipcc cross-compiles).

Its matrix instructions are asm statements: the compiler neither knows that they are matrix instructions nor puts the wait
states between one and a reader of its result.  So nothing but the MFMAs may touch a chunk sum before the wait states behind the loop: no
spill, no move between the register files and no copy of a register that an MFMA of the loop has written.  And what
test_resident_codegen checks of k_resident: nothing but the copies' own set-ups names M0, no `vmcnt` wait in the loop but the hand-written ones."""
import re
import shutil

import pytest

INSTANCE = re.compile(r"^(_ZN12_GLOBAL__N_110k_extendedILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)EEEv\w+):(.*?)^\.Lfunc_end", re.S | re.M)
INSTANCES = 38

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def registers(operand):
    """numbers of the vector registers in v5, v[4:7] (accumulation registers: offset by 1000)"""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    lo, hi = (int(m.group(2)),) * 2 if m.group(2) else (int(m.group(3)), int(m.group(4)))
    return {n + (1000 if m.group(1) == "a" else 0) for n in range(lo, hi + 1)}


def test_every_instance(resident_assembly):
    seen = 0
    for text in resident_assembly.values():
        for m in INSTANCE.finditer(text):
            name, (k, r, ta, tb, depth) = m.group(1), map(int, m.groups()[1:6])
            what = (k, r, 32 * ta, 32 * tb)
            lines = m.group(7).split("\n")
            mfma = [i for i, line in enumerate(lines) if "v_mfma_i32_16x16x64_i8" in line]
            assert len(mfma) == k * (k + 1) // 2 * ta * tb, what
            sums = set()
            for i in mfma:
                d, _, _, c = lines[i].split(";")[0].split("v_mfma_i32_16x16x64_i8")[1].split(", ")
                assert d.strip() == c.strip() and len(registers(d)) == 4, (what, lines[i])
                sums |= registers(d)
            assert len(sums) == sum((g - 1 + r - 1) // r for g in range(2, k + 2)) * ta * tb * 4, what
            end = next(i for i in range(mfma[-1], len(lines)) if "s_nop 15" in lines[i])
            by_hand, m0 = False, 0
            for i, line in enumerate(lines):
                if "#ASMSTART" in line or "#ASMEND" in line:
                    by_hand = "#ASMSTART" in line
                    continue
                code = line.split(";")[0].strip()
                if re.search(r"\bm0\b", code):
                    assert by_hand and code.startswith("s_add_u32 m0,"), (what, line)
                    m0 += 1
                if mfma[0] <= i <= end and code and "v_mfma" not in code:
                    assert by_hand or "vmcnt" not in code, (what, line)
                    assert not re.search(r"v_accvgpr|scratch_|buffer_", code), (what, line)
                    used = set().union(*(registers(x) for x in re.split(r"[ ,]+", code)))
                    assert not used & sums, (what, line)
            assert m0 >= k, what
            at = text.index(".name:           " + name)
            about = text[text.rindex("- .agpr_count", 0, at):text.find("- .agpr_count", at)]
            for key in ("private_segment_fixed_size", "vgpr_spill_count", "sgpr_spill_count"):
                assert re.search(r"\.%s:\s+(\d+)" % key, about).group(1) == "0", (what, key)
            seen += 1
    assert seen == INSTANCES
