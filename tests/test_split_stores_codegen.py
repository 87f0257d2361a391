"""Code-generation checks of the split's stores (CPU only: hipcc cross-compiles): the 16-byte ones written as asm statements bring the wait
states of their own that nobody else adds, and columns with one scale per slice go out in whole chunks."""
import re
import shutil
import subprocess

import pytest

from test_split_codegen import FLAGS, SRC

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("assembly") / "split.s")
    pr = subprocess.run(["hipcc", *FLAGS, "--cuda-device-only", "-S", SRC, "-o", out],
                        stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert pr.returncode == 0, pr.stdout[-3000:]
    return open(out).read()


def wait_states(instruction):
    m = re.match(r"s_nop (\d+)", instruction)
    return int(m.group(1)) + 1 if m else 1


def test_wide_stores_by_hand_bring_their_wait_states(assembly):
    # A vector instruction may write a register of a store of more than 8 bytes from the third wait state on.  The compiler sees no store in an asm
    # statement and keeps no distance, so the two states have to be in the statement, whatever comes behind it.
    seen, short = 0, []
    for m in re.finditer(r"#ASMSTART(.*?)#ASMEND", assembly, re.S):
        code = [x for x in (line.split(";")[0].strip() for line in m.group(1).split("\n")) if x]
        for i, x in enumerate(code):
            if re.match(r"(global|flat|buffer|scratch)_store_\w*x[34]\b", x):
                seen += 1
                if sum(wait_states(y) for y in code[i + 1:]) < 2:
                    short.append(code)
    assert seen > 0 and not short, (seen, short[:1], len(short))


def test_columns_of_one_scale_per_slice_go_out_in_whole_chunks(assembly):
    # Slices are written through L2, each store by itself: a column's 16 consecutive bytes in stores of 4 would go through as four pieces.
    seen = 0
    for m in re.finditer(r"^(_Z\S*k_split_psILi\d+ELi(\d+)ELi\d+EE\S*):(.*?)^\.Lfunc_end", assembly, re.S | re.M):
        seen += 1
        through = re.findall(r"\t(global_store_\w+) .* sc1", m.group(3))
        u = int(m.group(2))                              # chunks a thread holds of a column, four quads of a row instead
        assert through.count("global_store_dwordx4") >= u and through.count("global_store_dword") <= 4 * u, (m.group(1), through)
        assert set(through) == {"global_store_dwordx4", "global_store_dword"}, (m.group(1), through)
    assert seen == 6
