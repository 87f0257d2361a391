"""What the generated code of the kernels with resident chunk sums (csrc/ozimmu_resident.hip) has to look like; build() looks at
the assembly of every instance before it links the library.

Two things in these kernels rest on what the compiler does with asm statements that it does not look into:
  * their copies into LDS: M0 holds the LDS address, set by the first copy of a slice and relied on by the others, and hand-written
    `s_waitcnt vmcnt(N)` count the copies in flight.  So nothing else in the kernel may name M0, and the loop holds neither
    spills (whose reloads bring waits of their own) nor moves to and from accumulation registers nor a `vmcnt` wait of the compiler's;
  * the matrix instructions of the kernels that add in place (k_extended, k_held and their like): the compiler neither knows that they are matrix
    instructions nor puts the wait states before and behind them.  So nothing but they may touch a chunk sum before the wait states behind
    the loop (no spill, no move between the register files, no copy), and no ordinary vector instruction may write an operand of one
    within the two wait states before it."""
from __future__ import annotations

import re

MFMA = "v_mfma_i32_16x16x64_i8"
HELD_KS = range(5, 15)      # slice counts with tiles that hold slices of A (k_held)
OPERAND_WAIT_STATES = 2     # between a vector instruction that writes a register and a matrix instruction that reads it
KERNEL = re.compile(r"^(_ZN12_GLOBAL__N_1\d+(k_resident|k_cut|k_extended|k_held|k_per_slice)I((?:L[ib]\d+E)+)EEv\w+):(.*?)^\.Lfunc_end", re.S | re.M)


def registers(operand: str) -> set:
    """numbers of the vector registers in v5, v[4:7] (accumulation registers: offset by 1000)"""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    lo, hi = (int(m.group(2)),) * 2 if m.group(2) else (int(m.group(3)), int(m.group(4)))
    return {n + (1000 if m.group(1) == "a" else 0) for n in range(lo, hi + 1)}


def num_chunks(k: int, r: int) -> int:
    return sum((g - 1 + r - 1) // r for g in range(2, k + 2))


class Wrong(RuntimeError):
    pass


def _require(ok, *what):
    if not ok:
        raise Wrong(f"generated code: {what}")


def written_by_vector_instruction(code: str) -> set:
    """registers that an ordinary vector instruction (no matrix instruction, no memory access) writes"""
    name, _, rest = code.partition(" ")
    if not name.startswith("v_") or name.startswith(("v_mfma", "v_cmp", "v_nop")):
        return set()
    return registers(rest.split(",")[0])


def _wait_states(code: str) -> int:
    m = re.match(r"s_nop (\d+)", code)
    return int(m.group(1)) + 1 if m else 1


def check_operands(lines: list, what: tuple) -> None:
    """No ordinary vector instruction writes an operand of a matrix instruction within the wait states before it, on any way there:
    the instructions above it, and where one of those is a loop's label also the ones above the branch back to it."""
    code = [line.split(";")[0].strip() for line in lines]
    code = [c for c in code if c and not (c.startswith(".") and not c.startswith(".LBB"))]
    at_branch = {}
    for i, c in enumerate(code):
        m = re.match(r"s_c?branch\w* (\.LBB\w+)", c)
        if m:
            at_branch.setdefault(m.group(1) + ":", []).append(i)

    def look(i, states, used, mfma):
        while i >= 0 and states < OPERAND_WAIT_STATES:
            c = code[i]
            if c.startswith(".LBB"):
                for j in at_branch.get(c, []):
                    look(j, states, used, mfma)
                i -= 1
                continue
            if c.startswith("s_branch"):
                return                       # (not reached from above)
            _require(not written_by_vector_instruction(c) & used, what, c, mfma)
            states += _wait_states(c)
            i -= 1

    for i, c in enumerate(code):
        if c.startswith(MFMA):
            used = set().union(*(registers(x) for x in c[len(MFMA):].split(",")[1:]))
            look(i - 1, 0, used, c)


def check_body(body: str, k: int, r: int, ta: int, tb: int, in_place: bool, what: tuple) -> None:
    lines = body.split("\n")
    mfma = [i for i, line in enumerate(lines) if MFMA in line]
    _require(len(mfma) == k * (k + 1) // 2 * ta * tb, what, "matrix instructions", len(mfma))
    sums, end = set(), mfma[-1]
    if in_place:
        for i in mfma:
            d, _, _, c = lines[i].split(";")[0].split(MFMA)[1].split(", ")
            _require(d.strip() == c.strip() and len(registers(d)) == 4, what, lines[i])
            sums |= registers(d)
        _require(len(sums) == num_chunks(k, r) * ta * tb * 4, what, "chunk sums", len(sums))
        nops = [i for i in range(mfma[-1], len(lines)) if "s_nop 15" in lines[i]]
        _require(len(nops) >= 2, what, "no wait states behind the loop")
        end = nops[1]
        check_operands(lines, what)
    by_hand, m0 = False, 0
    for i, line in enumerate(lines):
        if "#ASMSTART" in line or "#ASMEND" in line:
            by_hand = "#ASMSTART" in line
            continue
        code = line.split(";")[0].strip()
        if re.search(r"\bm0\b", code):
            _require(by_hand and code.startswith("s_add_u32 m0,"), what, line)
            m0 += 1
        if mfma[0] <= i <= end and code and MFMA not in code:
            _require(by_hand or "vmcnt" not in code, what, line)
            _require(not re.search(r"v_accvgpr|scratch_|buffer_", code), what, line)
            if in_place:
                _require(not set().union(*(registers(x) for x in re.split(r"[ ,]+", code))) & sums, what, line)
    _require(m0 >= k, what, "copies' own set-ups of M0", m0)


def check_lanes(body: str, ta: int, tb: int, what: tuple) -> None:
    """k_held's pieces that four waves share: half of the lanes are off for one copy, and on again in the same asm statement."""
    halves = 0
    for statement in re.findall(r"#ASMSTART(.*?)#ASMEND", body, re.S):
        code = [c for c in (line.split(";")[0].strip() for line in statement.split("\n")) if c]
        off = [i for i, c in enumerate(code) if re.match(r"s_\w+ exec\b", c)]
        if not off:
            continue
        _require(len(off) == 2 and off[1] == off[0] + 2 and code[off[0]].startswith("s_mov_b64 exec, s[")
                 and code[off[0] + 1].startswith("global_load_lds_dwordx4") and code[off[1]] == "s_mov_b64 exec, -1", what, code)
        halves += 1
    _require((halves > 0) == (ta % 2 == 1 or tb % 2 == 1), what, "copies with half of the lanes", halves)


def check_kernels(text: str, k: int) -> dict:
    """Looks at every kernel in the assembly of ozimmu_resident.hip compiled for k slices; raises Wrong, also where a kind that has to be
    there is missing.  Returns how many there are of each kind."""
    seen = dict.fromkeys(("k_resident", "k_cut", "k_extended", "k_held", "k_per_slice"), 0)
    for m in KERNEL.finditer(text):
        name, kind, args = m.group(1), m.group(2), [int(x) for x in re.findall(r"L[ib](\d+)E", m.group(3))]
        what = (kind, *args)
        if kind == "k_per_slice":
            kk, ta, tb, _, _, in_place = args
            r = 1
        else:
            kk, r, ta, tb = args[:4]
            in_place = kind in ("k_extended", "k_held")
        _require(kk == k, what)
        check_body(m.group(4), k, r, ta, tb, bool(in_place), what)
        if kind == "k_held":
            check_lanes(m.group(4), ta, tb, what)
        at = text.index(".name:           " + name)
        about = text[text.rindex("- .agpr_count", 0, at):text.find("- .agpr_count", at)]
        for key in ("private_segment_fixed_size", "vgpr_spill_count", "sgpr_spill_count"):
            _require(re.search(r"\.%s:\s+(\d+)" % key, about).group(1) == "0", what, key)
        seen[kind] += 1
    # (one that KERNEL no longer matches would be linked without a look)
    for kind in ("k_resident", "k_cut", *(("k_held",) if k in HELD_KS else ())):
        _require(seen[kind] > 0, k, "no", kind, "in the assembly")
    return seen


def check_resident(text: str, k: int) -> dict:
    """check_kernels, which looks at k_held too, with the counts of the others."""
    return {kind: count for kind, count in check_kernels(text, k).items() if kind != "k_held"}
