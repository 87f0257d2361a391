"""Code-generation check of the split with one scale per slice (CPU only: hipcc cross-compiles): what a thread holds of a vector
stays in registers.  Spilled, the elements go to memory and back for every slice, which is what keeping them was to avoid."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "paper_2409_13313_amd", "csrc", "ozimmu_split.hip")
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument"]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_nothing_is_spilled(tmp_path):
    out = str(tmp_path / "split.s")
    pr = subprocess.run(["hipcc", *FLAGS, "--cuda-device-only", "-S", SRC, "-o", out],
                        stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert pr.returncode == 0, pr.stdout[-3000:]
    spilled, seen = [], 0
    for m in re.finditer(r"- \.agpr_count:(.*?)\.wavefront_size", open(out).read(), re.S):
        name = re.search(r"\.name:\s+(\S+)", m.group(1)).group(1)
        if "k_split_ps" not in name:
            continue
        seen += 1
        if re.search(r"\.(?:vgpr|sgpr)_spill_count:\s+[1-9]|\.private_segment_fixed_size:\s+[1-9]", m.group(1)):
            spilled.append(name)
    assert seen == 6 and not spilled, spilled
