"""Build the HIP library (gfx950 only) in-tree: csrc/*.hip -> libozimmu.so."""
from __future__ import annotations

import glob
import importlib.util
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libozimmu.so")
SOURCES = ["ozimmu_api.hip", "ozimmu_split.hip", "ozimmu_gemm.hip"]
# ozimmu_resident.hip holds kernels specialised for a slice count: one compilation per count, all of them linked into
# the object of the chunk GEMM (whoever links that object gets every way to run the schedule)
RESIDENT_KS = range(3, 17)
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument"]


def _codegen():
    """codegen.py, without the package (whose import needs the library)"""
    spec = importlib.util.spec_from_file_location("ozimmu_codegen", os.path.join(HERE, "codegen.py"))
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


def build(verbose: bool = False) -> str:
    """Compile every source and link the shared library; always recompiles.  The assembly of the kernels whose asm statements the
    compiler does not look into (codegen.py) is checked on the way: no library comes of code that fails."""
    codegen = _codegen()
    objs = [os.path.join(CSRC, src.replace(".hip", ".o")) for src in SOURCES]
    core = os.path.join(CSRC, "ozimmu_gemm_core.o")
    resident = [os.path.join(CSRC, f"ozimmu_resident_k{k}.o") for k in RESIDENT_KS]
    jobs = [(src, [], core if obj.endswith("ozimmu_gemm.o") else obj) for src, obj in zip(SOURCES, objs)]
    jobs += [("ozimmu_resident.hip", [f"-DOZ_RES_K={k}"], obj) for k, obj in zip(RESIDENT_KS, resident)]

    def compile_one(job):
        src, defs, obj = job
        with tempfile.TemporaryDirectory() as tmp:
            # (the assembly that becomes the object is kept beside it for a look)
            made = os.path.join(tmp, os.path.basename(obj))
            cmd = ["hipcc", *FLAGS, *defs, *(["--save-temps=obj"] if defs else []), "-c", os.path.join(CSRC, src), "-o", made]
            if verbose:
                print(" ".join(cmd), flush=True)
            pr = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
            out = "\n".join(l for l in pr.stdout.splitlines() if "packed-fp32-ops" not in l)
            if pr.returncode != 0:
                raise RuntimeError(f"hipcc failed: {' '.join(cmd)}\n{out}")
            if verbose and out.strip():
                print(out)
            if defs:
                text, = (open(f).read() for f in glob.glob(os.path.join(tmp, "*gfx950*.s")))
                seen = codegen.check_resident(text, int(defs[0].split("=")[1]))
                if not all(seen[kind] for kind in ("k_resident", "k_cut")):
                    raise RuntimeError(f"{defs[0]}: kernels missing from the assembly: {seen}")
            shutil.copyfile(made, obj)

    with ThreadPoolExecutor(max_workers=8) as pool:
        list(pool.map(compile_one, jobs))
    subprocess.run(["ld", "-r", "-o", os.path.join(CSRC, "ozimmu_gemm.o"), core, *resident], check=True)
    cmd = ["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    subprocess.run(cmd, check=True)
    return LIB


def build_single(source: str, lib: str) -> str:
    """One-file shared library with the same flags (bench.py's measurement probe is built this way)."""
    cmd = ["hipcc", *FLAGS, "-shared", source, "-o", lib]
    pr = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if pr.returncode != 0:
        raise RuntimeError(f"hipcc failed: {' '.join(cmd)}\n{pr.stdout}")
    return lib


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
