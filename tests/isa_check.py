"""Static check of the compiled bf16 attention kernel's ISA.

The matrix phase of the kernel issues its MFMAs through inline asm, so the compiler does not know
that the registers those statements write are matrix-pipe results: it inserts no wait states if
it decides to read, copy or overwrite one of them with a vector instruction right behind the
MFMA.  Behind the last step of a unit the kernel waits by hand; behind the chains of the others it relies on
what follows being long enough: the scores are finished by the MFMAs behind them, the output tile is next touched
at the end of the vector phase, with a barrier and branches in between.  This check makes sure that it is, and that the compiler
did not add an access of its own.

Rule checked: a vector register written by a `v_mfma` is not named by any non-MFMA instruction
within WAIT_STATES wait states (one per issued instruction, N + 1 for `s_nop N`) after it, in straight-line
code (mfma_hazards) and on every path through branches, loops and barriers (flow_hazards).  (An MFMA that accumulates into
the same registers is interlocked by hardware.)
The 32x32x16 bf16 MFMA has 8 passes; the compiler's own rule for it is 11 wait states."""
from __future__ import annotations

import os
import re
import subprocess
import tempfile

from paper_2507_09071_amd import build as _build

WAIT_STATES = 12
OPERAND_WAIT_STATES = 2   # vector write of a register, MFMA that reads it
KERNELS = ("_ZN2bs17attn_prefill_bf16ILi128EEE", "_ZN2bs17attn_prefill_bf16ILi64EEE")


def compile_to_isa(out_path: str) -> None:
    cmd = [_build.hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-falign-loops=64",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
           "-I", os.path.join(_build.ROOT, "include"), "-I", _build.CSRC,
           *os.environ.get("BS_EXTRA_HIPCC_FLAGS", "").split(),
           "--cuda-device-only", "-S", os.path.join(_build.CSRC, "attn_prefill.hip"), "-o", out_path]
    subprocess.run(cmd, check=True, capture_output=True)


def _regs(text: str) -> set:
    out = set()
    for m in re.finditer(r"v\[(\d+):(\d+)\]", text):
        out.update(range(int(m.group(1)), int(m.group(2)) + 1))
    for m in re.finditer(r"(?<![\w\[])v(\d+)\b", text):
        out.add(int(m.group(1)))
    return out


def kernel_instructions(isa: str, symbol_prefix: str) -> list:
    start = isa.index(symbol_prefix)
    end = isa.index("s_endpgm", start)
    ins = []
    for line in isa[start:end].split("\n"):
        t = line.split(";")[0].strip()
        if t and not t.startswith(".") and not t.endswith(":"):
            ins.append(t)
    return ins


def mfma_hazards(ins: list) -> list:
    """List of (mfma, wait states, offending instruction)."""
    found = []
    for a, t in enumerate(ins):
        if not t.startswith("v_mfma"):
            continue
        dst = _regs(t.split(",")[0])
        ws = 0
        for u in ins[a + 1:a + 1 + 4 * WAIT_STATES]:
            if u.startswith(("s_cbranch", "s_branch", "s_barrier", "s_endpgm")):
                break   # the rule is checked in straight-line code only
            if u.startswith("v_mfma"):
                ws += 1
            else:
                if _regs(u) & dst:
                    found.append((t, ws, u))
                m = re.match(r"s_nop (\d+)", u)
                ws += int(m.group(1)) + 1 if m else 1
            if ws >= WAIT_STATES:
                break
    return found


def lds_read_hazards(ins: list) -> list:
    """The operand reads of the matrix phase are asm `ds_read_b128` waited for by hand-counted
    `s_waitcnt lgkmcnt(N)`.  The compiler believes the destination holds the value as soon as
    the asm statement is over; check that nothing names a destination register while its read
    may still be in flight.  LDS reads complete in order: after `lgkmcnt(N)` all but the N
    youngest are done (scalar loads share the counter and only make the wait stricter).
    Straight-line code only: the list of reads in flight is dropped at branches and barriers; flow_hazards
    follows those that cross one (the walk's branches stand between two batches).  Returns (read, offending
    instruction) pairs."""
    found = []
    inflight = []   # (instruction, destination registers), oldest first
    for t in ins:
        if t.startswith(("s_cbranch", "s_branch", "s_barrier", "s_endpgm")):
            inflight = []
            continue
        m = re.match(r"s_waitcnt .*lgkmcnt\((\d+)\)", t)
        if m:
            n = int(m.group(1))
            inflight = inflight[len(inflight) - n:] if n else []
            continue
        if t.startswith("s_waitcnt") and "lgkmcnt" not in t and "vmcnt" not in t:
            inflight = []   # a bare immediate: treat as a full wait only if it names no counter
            continue
        named = _regs(t)
        for r, dst in inflight:
            if named & dst:
                found.append((r, t))
        if t.startswith("ds_read"):
            inflight.append((t, _regs(t.split(",")[0])))
    return found


def operand_hazards(ins: list) -> list:
    """List of (vector instruction, mfma): an operand of an MFMA written by a vector instruction less than
    OPERAND_WAIT_STATES wait states before it.  The hardware does not interlock that and the compiler, which sees no
    matrix instruction, does not keep the distance.  A conditional branch is a wait state like any instruction: the code
    behind it follows if it is not taken."""
    found = []
    for a, t in enumerate(ins):
        if not t.startswith("v_") or t.startswith(("v_mfma", "v_cmp", "v_readlane", "v_readfirstlane")):
            continue
        operands = t.split(",")
        dst, ws = _regs(operands[0]), 0
        if "swap" in t.split()[0]:
            dst |= _regs(operands[1])   # writes both
        for u in ins[a + 1:a + 1 + 2 * OPERAND_WAIT_STATES]:
            if u.startswith(("s_branch", "s_endpgm")) or ws >= OPERAND_WAIT_STATES:
                break
            if u.startswith("v_mfma"):
                if _regs(u.split(",", 1)[1]) & dst:
                    found.append((t, u))
                break
            m = re.match(r"s_nop (\d+)", u)
            ws += int(m.group(1)) + 1 if m else 1
    return found


def kernel_blocks(isa: str, symbol_prefix: str) -> list:
    """The kernel's basic blocks: [(instructions, indices of the blocks that may follow)].  An instruction of an inline asm statement
    has a leading "asm "."""
    start = isa.index("\n" + symbol_prefix) + 1
    end = isa.index(".Lfunc_end", start)
    blocks, label_at, in_asm = [[]], {}, False
    for line in isa[start:end].split("\n"):
        if "#ASMSTART" in line or "#ASMEND" in line:
            in_asm = "#ASMSTART" in line
            continue
        t = line.split(";")[0].strip()
        if t.endswith(":"):
            if blocks[-1]:
                blocks.append([])
            label_at[t[:-1]] = len(blocks) - 1
        elif t and not t.startswith("."):
            blocks[-1].append(("asm " if in_asm else "") + t)
            if t.startswith(("s_cbranch", "s_branch", "s_endpgm")):
                blocks.append([])
    out = []
    for i, ins in enumerate(blocks):
        last = ins[-1] if ins else ""
        follow = [label_at[last.split()[1]]] if last.startswith(("s_cbranch", "s_branch")) else []
        if not last.startswith(("s_branch", "s_endpgm")) and i + 1 < len(blocks):
            follow.append(i + 1)
        out.append((ins, follow))
    return out


def _wait_states(t: str) -> int:
    m = re.match(r"s_nop (\d+)", t)
    return int(m.group(1)) + 1 if m else 1


def flow_hazards(blocks: list) -> list:
    """The rules for MFMA results, their operands and asm LDS reads on every path through the kernel.  Along a path every register that an
    MFMA (a vector instruction) has written has so many wait states left in which no other instruction may name it (no MFMA may read it);
    LDS operations in flight are known by how many were issued behind them, as they complete in order.  Where paths meet, the longer wait
    and the reads of both count.  Returns (rule, instruction, register)."""
    found = set()

    def run(ins, state):
        result, operand, reads = dict(state[0]), dict(state[1]), dict(state[2])
        for t in ins:
            from_asm, u = t.startswith("asm "), t[4:] if t.startswith("asm ") else t
            operands = u.split(None, 1)[1].split(", ") if " " in u else []
            is_mfma, named = u.startswith("v_mfma"), _regs(u)
            if is_mfma:
                sources = _regs(", ".join(operands[1:3]))   # (the accumulator is interlocked)
                found.update(("result as operand", u, r) for r in sources & result.keys())
                found.update(("operand", u, r) for r in _regs(", ".join(operands[1:])) & operand.keys())
            else:
                found.update(("result", u, r) for r in named & result.keys())
            found.update(("LDS read in flight", u, r) for r in named & reads.keys())
            m = re.match(r"s_waitcnt .*lgkmcnt\((\d+)\)", u)
            if m:
                reads = {r: behind for r, behind in reads.items() if behind < int(m.group(1))}
            if u.startswith("ds_"):
                reads = {r: behind + 1 for r, behind in reads.items()}
                if from_asm and u.startswith("ds_read"):
                    reads.update((r, 0) for r in _regs(operands[0]))   # (a read of the compiler's own is waited for by the compiler)
            ws = _wait_states(u)
            for left in (result, operand):
                for r in [r for r in left if left[r] <= ws]:
                    del left[r]
                for r in left:
                    left[r] -= ws
            if is_mfma:
                result.update((r, WAIT_STATES) for r in _regs(operands[0]))
                for r in _regs(operands[0]):
                    operand.pop(r, None)
            elif u.startswith("v_") and not u.startswith(("v_cmp", "v_readlane", "v_readfirstlane")):
                operand.update((r, OPERAND_WAIT_STATES) for r in _regs(operands[0]) | (_regs(operands[1]) if "swap" in u.split()[0] else set()))
        return result, operand, reads

    meet = (max, max, min)   # (fewer operations behind a read: a wait for a given number of them ends later)
    entry = [None] * len(blocks)
    entry[0] = ({}, {}, {})
    todo = [0]
    while todo:
        i = todo.pop()
        state = run(blocks[i][0], entry[i])
        for j in blocks[i][1]:
            merged = entry[j] and tuple({r: f(x[r] for x in (a, b) if r in x) for r in a.keys() | b.keys()} for f, a, b in zip(meet, entry[j], state))
            if entry[j] is None or merged != entry[j]:
                entry[j] = merged or state
                todo.append(j)
    return sorted(found, key=str)


def check(isa_path: str | None = None) -> dict:
    """Compile (unless a listing is given) and return {kernel symbol prefix: [hazards]}."""
    if isa_path is None:
        with tempfile.TemporaryDirectory() as d:
            isa_path = os.path.join(d, "attn_prefill.s")
            compile_to_isa(isa_path)
            isa = open(isa_path).read()
    else:
        isa = open(isa_path).read()
    out = {}
    for k in KERNELS:
        ins = kernel_instructions(isa, k)
        out[k] = mfma_hazards(ins) + lds_read_hazards(ins) + operand_hazards(ins) + flow_hazards(kernel_blocks(isa, k))
    return out


if __name__ == "__main__":
    res = check()
    for k, h in res.items():
        print(k, "hazards:", len(h))
        for item in h[:10]:
            print("  ", *[str(x)[:70] for x in item])
    raise SystemExit(1 if any(res.values()) else 0)
