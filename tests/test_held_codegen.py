"""The assembly of every instance of k_held (CPU only: hipcc cross-compiles): sums that nothing but its matrix instructions touches, no spill,
nothing but the copies' own set-ups names M0 (codegen.py, which the build runs too)."""
import shutil

import pytest

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def test_every_instance(resident_assembly):
    from paper_2409_13313_amd import codegen
    seen = {k: codegen.check_kernels(text, k)["k_held"] for k, text in resident_assembly.items()}
    assert sum(seen.values()) == 20 and all(seen[k] > 0 for k in range(5, 15)), seen
    for k, text in resident_assembly.items():
        for m in codegen.KERNEL.finditer(text):
            if m.group(2) == "k_held":
                # lanes are switched off for half copies only, and on again in the same statement
                lines = [line.strip() for line in m.group(4).split("\n")]
                off = [i for i, line in enumerate(lines) if line.startswith("s_mov_b64 exec, s[")]
                assert all(lines[i + 1].startswith("global_load_lds_dwordx4") and lines[i + 2] == "s_mov_b64 exec, -1" for i in off), m.group(1)
