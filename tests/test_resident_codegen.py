"""Code-generation checks of the kernel with resident chunk sums, every instance of it (CPU only: hipcc cross-compiles).

Its copies into LDS are inline assembly that the compiler does not follow: M0 holds their LDS address, and hand-written
`s_waitcnt vmcnt(N)` count the copies in flight.  The first copy of a slice sets M0
and the others rely on it, so nothing else in the whole kernel may name it; and the loop holds neither spills (whose reloads
bring waits of their own) nor moves to and from accumulation registers nor a `vmcnt` wait of the compiler's."""
import re
import shutil

import pytest

INSTANCE = re.compile(r"^(_ZN12_GLOBAL__N_110k_residentILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)EEEv\w+):(.*?)^\.Lfunc_end", re.S | re.M)

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


def test_every_instance(resident_assembly):
    seen = 0
    for text in resident_assembly.values():
        for m in INSTANCE.finditer(text):
            name, (k, r, ta, tb, depth, waves) = m.group(1), map(int, m.groups()[1:7])
            what = (k, r, 32 * ta, 32 * tb)
            lines = m.group(8).split("\n")
            mfma = [i for i, line in enumerate(lines) if "v_mfma_i32_16x16x64_i8" in line]
            assert len(mfma) == k * (k + 1) // 2 * ta * tb, what
            by_hand = False
            m0 = 0
            for i, line in enumerate(lines):
                if "#ASMSTART" in line or "#ASMEND" in line:
                    by_hand = "#ASMSTART" in line
                    continue
                code = line.split(";")[0]
                if re.search(r"\bm0\b", code):
                    assert by_hand and code.strip().startswith("s_add_u32 m0,"), (what, line)
                    m0 += 1
                if mfma[0] <= i <= mfma[-1]:
                    assert by_hand or "vmcnt" not in code, (what, line)
                    assert not re.search(r"v_accvgpr|scratch_|buffer_", code), (what, line)
            assert m0 >= k, what
            # one exponent per row and column is all that this kernel adds its sums up with: term by term (an ldexp for every
            # sum), or scaled (one for every element of a tile).  A third way, or one of them twice, costs every call (twice
            # only where registers are short, for stores that stay in L2 and others)
            w = sum((g - 1 + r - 1) // r for g in range(2, k + 2))
            ends = w + 1 if w * ta * tb < (60 if waves == 1 else 32) else w + 2
            ldexps = sum("v_ldexp_f64" in line for line in lines)
            assert ldexps <= 4 * ta * tb * ends + 2, (what, ldexps)
            stores = [line for line in lines if "_store_dwordx2" in line]
            assert len(stores) == 4 * ta * tb * (4 if ends == w + 1 else 3), (what, len(stores))
            assert sum(" nt" in line for line in stores) == 8 * ta * tb, what      # (no two of them merged into one)
            at = text.index(".name:           " + name)
            about = text[text.rindex("- .agpr_count", 0, at):text.find("- .agpr_count", at)]
            for key in ("private_segment_fixed_size", "vgpr_spill_count", "sgpr_spill_count"):
                assert re.search(r"\.%s:\s+(\d+)" % key, about).group(1) == "0", (what, key)
            seen += 1
    assert seen == 196
