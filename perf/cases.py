"""What a user of this framework has it do, as cases that can be timed and compared.

Every case is one FP64 matrix product D = A B (or C <- alpha op(A) op(B) + beta C) emulated with k INT8 slices,
through the entry points of paper_2409_13313_amd.ozimmu.  A is m x n, B is n x p: n is the inner dimension.
Inputs are the random matrices of the method's own experiments, (U - 0.5) exp(phi N) with U uniform and N normal.

A case holds
  call       "dgemm", "gemm_ex" (transposes, alpha, beta), "variant" (split / accumulate mode) or "static" (the
             library's own workspace)
  m, n, p, k, phi
  workspace  dgemm and variant: "kept" (output and workspace laid out once, as a solver's inner loop or a benchmark
             does) or "per call" (neither is handed over, the binding allocates both)
  pad        extra elements between the rows of A, B and the output (views into larger arrays)
"""
from __future__ import annotations

import math

import torch

from paper_2409_13313_amd import ozimmu


def listed():
    return [
        # the smallest call of the benchmark list: launches and latency
        {"name": "square-256", "call": "dgemm", "m": 256, "n": 256, "p": 256, "k": 8, "phi": 0.5,
         "workspace": "kept", "pad": 0},
        # an odd small block, as a factorisation's update has it, without a workspace to hand over (no allocation allowed)
        {"name": "static-ragged", "call": "static", "m": 777, "n": 1001, "p": 513, "k": 7, "phi": 1.0, "pad": 3},
        # the accuracy sweep's matrix, with the slice count that matches native FP64 at phi = 2
        {"name": "square-1024-k9", "call": "dgemm", "m": 1024, "n": 1024, "p": 1024, "k": 9, "phi": 2.0,
         "workspace": "kept", "pad": 0},
        # few output tiles, longer inner dimension (Gram matrices, projections)
        {"name": "long-1024x16384", "call": "dgemm", "m": 1024, "n": 16384, "p": 1024, "k": 8, "phi": 0.5,
         "workspace": "kept", "pad": 0},
        # the GEMM routine with everything on: both operands transposed, alpha, beta, ragged sizes, no workspace given
        {"name": "gemm-ex-ragged", "call": "gemm_ex", "m": 1537, "n": 2051, "p": 1283, "k": 9, "phi": 1.0,
         "transA": True, "transB": True, "alpha": -1.0, "beta": 0.5, "pad": 1},
        # an ordinary call with the simplest signature, sizes that no tile divides
        {"name": "plain-3000", "call": "dgemm", "m": 3000, "n": 2900, "p": 3100, "k": 8, "phi": 0.5,
         "workspace": "per call", "pad": 0},
        # throughput against accuracy at 4096, phi = 0
        {"name": "square-4096", "call": "dgemm", "m": 4096, "n": 4096, "p": 4096, "k": 8, "phi": 0.0,
         "workspace": "kept", "pad": 0},
        # the earlier method that the comparison of variants runs: bit-mask slices, one FP64 addition per slice pair
        {"name": "variant-ozimmu-4096", "call": "variant", "m": 4096, "n": 4096, "p": 4096, "k": 9, "phi": 1.0,
         "split": "bitmask", "accumulate": "per_pair", "workspace": "kept", "pad": 0},
        # large square product with few slices
        {"name": "square-8192-k6", "call": "dgemm", "m": 8192, "n": 8192, "p": 8192, "k": 6, "phi": 0.5,
         "workspace": "kept", "pad": 0},
        # long inner dimension: short chunks, thirty FP64 addends per element
        {"name": "long-4096x65536-k10", "call": "dgemm", "m": 4096, "n": 65536, "p": 4096, "k": 10, "phi": 1.0,
         "workspace": "kept", "pad": 0},
        # the headline workload
        {"name": "square-16384", "call": "dgemm", "m": 16384, "n": 16384, "p": 16384, "k": 8, "phi": 0.5,
         "workspace": "kept", "pad": 0},
        # the same size for inputs of wide exponent range, which need more slices
        {"name": "square-16384-k12", "call": "dgemm", "m": 16384, "n": 16384, "p": 16384, "k": 12, "phi": 4.0,
         "workspace": "kept", "pad": 0},
    ]


def _cost(c):
    """Integer operations of the slice products plus what the padding to whole tiles and the passes over memory weigh."""
    m, n, p = (-(-c[d] // 256) * 256 for d in ("m", "n", "p"))
    w = 4.0 if c["call"] == "variant" else 1.0   # one FP64 addition per pair, more passes over the operands
    return w * 2.0 * m * n * p * c["k"] * (c["k"] + 1) / 2


def draw(rng):
    """One more case: sizes by their logarithm over 32 .. 16384 (inner dimension to 65536), k = 3 .. 14."""
    limit = max(_cost(c) for c in listed() if c["call"] == "dgemm")

    def size(lo, hi):
        v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return v // 128 * 128 if v >= 512 and rng.random() < 0.4 else v

    while True:
        call = rng.choices(["dgemm", "gemm_ex", "variant", "static"], weights=[55, 20, 13, 12])[0]
        top = 1024 if call == "static" else 16384
        if rng.random() < 0.35:          # square, the usual case
            m = n = p = size(64, top)
        else:
            m, p = size(32, top), size(32, top)
            n = size(32, min(4 * top, 65536))
        c = {"call": call, "m": m, "n": n, "p": p, "k": rng.choice([3, 4, 5, 6, 7, 8, 8, 8, 9, 9, 10, 11, 12, 13, 14]),
             "phi": rng.choice([0.0, 0.5, 0.5, 1.0, 2.0, 4.0]), "pad": rng.choice([0, 0, 0, 1, 2])}
        if call in ("dgemm", "variant"):
            c["workspace"] = rng.choice(["kept", "kept", "per call"])
        if call == "gemm_ex":
            c["transA"], c["transB"] = rng.random() < 0.5, rng.random() < 0.5
            c["alpha"], c["beta"] = rng.choice([(1.0, 0.0), (-1.0, 0.5), (0.75, -0.25), (2.0, 0.0)])
        if call == "variant":
            c["split"], c["accumulate"] = rng.choice([("bitmask", "grouped"), ("bitmask", "per_pair"),
                                                      ("per_slice", "per_pair"), ("rn", "wide"), ("rn", "per_pair")])
        if _cost(c) > limit:
            continue
        if call == "static" and ozimmu.workspace_bytes_min(m, n, p, c["k"]) > ozimmu.STATIC_WORKSPACE_BYTES:
            continue
        return c


def _matrix(gen, rows, cols, phi, pad):
    full = torch.rand((rows, cols + pad), dtype=torch.float64, device="cuda", generator=gen).sub_(0.5)
    if phi:
        full.mul_(torch.randn((rows, cols + pad), dtype=torch.float64, device="cuda", generator=gen).mul_(phi).exp_())
    return full[:, :cols]


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    m, n, p, pad = c["m"], c["n"], c["p"], c["pad"]
    A = _matrix(gen, n, m, c["phi"], pad) if c.get("transA") else _matrix(gen, m, n, c["phi"], pad)
    B = _matrix(gen, p, n, c["phi"], pad) if c.get("transB") else _matrix(gen, n, p, c["phi"], pad)
    C = _matrix(gen, m, p, 0.0, pad) if c["call"] == "gemm_ex" else None
    return A, B, C


def prepare(case, seed):
    c = case
    A, B, C = _inputs(c, seed)
    state = {"case": c, "A": A, "B": B, "C": C, "D": None, "workspace": None}
    if c["call"] == "static" or c.get("workspace") == "kept":
        state["D"] = torch.empty((c["m"], c["p"] + c["pad"]), dtype=torch.float64, device="cuda")[:, :c["p"]]
    if c.get("workspace") == "kept":
        state["workspace"] = ozimmu.alloc_workspace(c["m"], c["n"], c["p"], c["k"], split=c.get("split", "rn"))
    return state


def run(state):
    c, A, B = state["case"], state["A"], state["B"]
    if c["call"] == "dgemm":
        return ozimmu.dgemm(A, B, c["k"], D=state["D"], workspace=state["workspace"])
    if c["call"] == "variant":
        return ozimmu.dgemm_variant(A, B, c["k"], c["split"], c["accumulate"], D=state["D"], workspace=state["workspace"])
    if c["call"] == "static":
        return ozimmu.dgemm_static(A, B, c["k"], state["D"])
    return ozimmu.gemm_ex(c["transA"], c["transB"], c["alpha"], A, B, c["beta"], state["C"], c["k"])


def work(case):
    m, n, p, k = (case[d] for d in ("m", "n", "p", "k"))
    old_c = m * p if case.get("beta") else 0
    return {"bytes": 8.0 * (m * n + n * p + m * p + old_c),          # FP64 in, FP64 out
            "flops": 2.0 * m * n * p * k * (k + 1) / 2}              # INT8 operations of the slice products that are kept


def tolerance(case):
    # The slices and the INT32 sums are integers, and the method fixes which FP64 additions are made and in which
    # order (one per chunk, after exact power-of-two scaling): every correct implementation gives the same bits.
    return "exact"


def exact(case, seed):
    # (the distance to this is the truncation after k slices, not a rounding error of the implementation)
    A, B, C = _inputs(case, seed)
    D = torch.mm(A.t() if case.get("transA") else A, B.t() if case.get("transB") else B)
    if case["call"] != "gemm_ex":
        return D
    return case["alpha"] * D + case["beta"] * C if case["beta"] else case["alpha"] * D
