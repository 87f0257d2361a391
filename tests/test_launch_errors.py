"""A kernel launch that fails is reported once, by the entry point that made it: left behind in the runtime it would be reported again by
whatever the caller launches next (the driver replaces the runtime's launch by one that fails; no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2409_13313_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_nothing_is_left_behind(tmp_path):
    objs = [os.path.join(CSRC, f) for f in ("ozimmu_split.o", "ozimmu_gemm.o")]
    if not all(os.path.exists(o) for o in objs):
        pytest.skip("library objects not built (run __graft_entry__.build())")
    drv, exe = str(tmp_path / "driver.o"), str(tmp_path / "driver")
    for cmd in (["hipcc", "-O1", "--offload-arch=gfx950", "-std=c++17", "-c", os.path.join(ROOT, "tests", "launch_error_driver.cpp"), "-o", drv],
                ["hipcc", "--offload-arch=gfx950", drv, *objs, "-o", exe], [exe]):
        pr = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
        assert pr.returncode == 0, pr.stdout[-3000:]
    assert "launch error driver ok" in pr.stdout
