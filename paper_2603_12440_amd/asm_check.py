"""Reads the generated gfx950 assembly for what the compiler cannot see to: the kernels issue MFMAs and direct-to-LDS loads from
assembly statements, around which it puts no wait states.  Every check walks backwards from an instruction over all paths that
lead to it, loops and far jumps included."""
from __future__ import annotations

import re

_REG = re.compile(r"\b([avs])(?:\[(\d+):(\d+)\]|(\d+)\b)")
_FAR = re.compile(r"s_add_u32\s+\S+\s+\S+\s+\((\.?\w+)-")
_NO_FALL_THROUGH = ("s_branch", "s_endpgm", "s_setpc_b64", "s_trap")


def _registers(text: str) -> list:
    """(class, first, last) of every register operand."""
    return [(c, int(lo or one), int(hi or one)) for c, lo, hi, one in _REG.findall(text)]


def _meet(x, y) -> bool:
    return x[0] == y[0] and x[1] <= y[2] and y[1] <= x[2]


class Listing:
    """The instructions of a listing and which ones can run right before each."""

    def __init__(self, asm: str):
        self.text, self.line, self.asm = [], [], []            # asm: from an assembly statement
        labels, jumps, inside = {}, [], False
        for n, raw in enumerate(asm.split("\n"), 1):
            if "#ASM" in raw:
                inside = "#ASMSTART" in raw
                continue
            t = raw.split(";")[0].strip()
            if not t or t.startswith("//"):
                continue
            if t.endswith(":"):
                labels[t[:-1]] = len(self.text)
                continue
            if t[0] == ".":
                continue
            if t.startswith(("s_branch", "s_cbranch")):
                jumps.append((len(self.text), t.split()[1]))
            elif t.startswith("s_setpc"):                      # a jump beyond a branch's reach: pc + (label - here)
                for back in range(1, 4):
                    far = _FAR.match(self.text[-back]) if back <= len(self.text) else None
                    if far:
                        jumps.append((len(self.text), far.group(1)))
                        break
                else:
                    raise ValueError(f"line {n}: a jump whose target is not known: {t}")
            self.text.append(t)
            self.line.append(n)
            self.asm.append(inside)
        self.jumped_from = {}
        for i, label in jumps:
            self.jumped_from.setdefault(labels[label], []).append(i)

    def before(self, i: int, states: int):
        """(instruction, wait states between it and instruction i) for all that can run fewer than `states` states earlier."""
        nearest, todo = {}, [(i, 0)]
        while todo:
            at, far = todo.pop()
            prev = list(self.jumped_from.get(at, ()))
            if at > 0 and not self.text[at - 1].startswith(_NO_FALL_THROUGH):
                prev.append(at - 1)
            for j in prev:
                if nearest.get(j, states) <= far:
                    continue
                nearest[j] = far
                yield j, far
                t = self.text[j]
                next_far = far + (int(t.split()[1], 0) + 1 if t.startswith("s_nop") else 1)
                if next_far < states:
                    todo.append((j, next_far))

    def found(self, i: int, j: int, far: int) -> str:
        return f"{self.line[i]}: {self.text[i]}   ({far} wait states after line {self.line[j]}: {self.text[j]})"


def lds_load_hazards(asm, listing: Listing = None) -> list:
    """Direct-to-LDS loads whose scalar base address a vector-ALU instruction (a `v_readfirstlane`, most of all) wrote fewer than 5
    wait states earlier: a vector-memory instruction may not read a scalar register that soon."""
    k = listing or Listing(asm)
    bad = []
    for i, t in enumerate(k.text):
        if not t.startswith("global_load_lds"):
            continue
        base = [r for r in _registers(t) if r[0] == "s"]
        for j, far in k.before(i, 5):
            w = k.text[j]
            # (the destination; a carry or compare result may be the second operand)
            if w.startswith("v_") and any(_meet(r, b) for r in _registers(",".join(w.split(None, 1)[1].split(",")[:2 if "_co_" in w else 1]))
                                          for b in base):
                bad.append(k.found(i, j, far))
    return bad


# What a vector-ALU or memory instruction has to keep from the MFMA whose result it reads or overwrites: 19 wait states for the
# longest shapes the kernels use (16 passes).
MFMA_RESULT_STATES = 19


def accumulator_hazards(asm, listing: Listing = None) -> list:
    """Where the compiler's own register traffic is too close to an MFMA: an accumulator (and, for MFMAs in assembly statements, an
    operand) written by a vector-ALU instruction fewer than 2 wait states before the MFMA takes it; and, for those in assembly
    statements, an accumulator that any other instruction reads or writes fewer than 19 states after the MFMA wrote it.  The compiler moves accumulators where
    paths meet if copies of a loop body stand in the branches of a condition."""
    k = listing or Listing(asm)
    bad = []
    for i, t in enumerate(k.text):
        if t.startswith("v_mfma"):
            takes = _registers(t) if k.asm[i] else _registers(t.split(",")[0])
            for j, far in k.before(i, 2):
                w = k.text[j]
                if w.startswith("v_") and not w.startswith("v_mfma") and any(_meet(r, s) for r in _registers(w.split(",")[0]) for s in takes):
                    bad.append(k.found(i, j, far))
        elif " a" in t:
            uses = [r for r in _registers(t) if r[0] == "a"]
            if not uses:
                continue
            for j, far in k.before(i, MFMA_RESULT_STATES):
                if k.asm[j] and k.text[j].startswith("v_mfma") and any(_meet(_registers(k.text[j])[0], u) for u in uses):
                    bad.append(k.found(i, j, far))
    return bad
