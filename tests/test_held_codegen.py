"""The assembly of every instance of k_held (CPU only: hipcc cross-compiles): sums that nothing but its matrix instructions touches, no spill,
nothing but the copies' own set-ups names M0, lanes off for half copies only (codegen.py, which the build runs too, and without a k_held makes no library)."""
import shutil

import pytest

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def test_every_instance(resident_assembly):
    from paper_2409_13313_amd import build, codegen
    seen = {k: codegen.check_resident(text, k)["k_held"] for k, text in resident_assembly.items()}
    assert sum(seen.values()) == 20 and all((seen[k] > 0) == (k in build.HELD_KS) for k in seen), seen
