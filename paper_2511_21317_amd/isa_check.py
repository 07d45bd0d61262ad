"""Checks the gfx950 assembly of this package's own kernels for what the compiler does not see: the wait states around
products (MFMA) that are written out as inline assembly.

For its own products the compiler keeps these distances itself; around an asm statement it keeps none.  So the build runs
hazards() over the assembly that the library is made of, and fails if there are any:
  * a vector instruction that writes an operand of such a product less than 2 wait states before it, or the lane mask less
    than 4 before it;
  * anything that touches a product's result less than 19 wait states behind it (what the longest product takes), but for a
    product that adds to the very same registers;
  * scratch memory in a kernel with such products (registers that are spilled are read and written at places of the
    compiler's choice).
An instruction counts as one wait state, `s_nop N` as N + 1.  Every path through the control flow is followed."""
from __future__ import annotations

import re

OPERAND_WAIT, EXEC_WAIT, RESULT_WAIT = 2, 4, 19

_REG = re.compile(r"\b([av])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _regs(text: str) -> frozenset:
    out = set()
    for kind, one, lo, hi in _REG.findall(text):
        out.update((kind, i) for i in (range(int(one), int(one) + 1) if one else range(int(lo), int(hi) + 1)))
    return frozenset(out)


class _Instr:
    __slots__ = ("op", "line", "args", "is_asm", "next", "prev")

    def __init__(self, line: str, is_asm: bool):
        self.line = line
        self.op, _, rest = line.partition(" ")
        self.args = [a.strip() for a in rest.split(",")] if rest else []
        self.is_asm = is_asm
        self.next, self.prev = [], []

    @property
    def states(self) -> int:
        return int(self.args[0], 0) + 1 if self.op == "s_nop" else 1

    @property
    def is_product(self) -> bool:
        return self.op.startswith(("v_mfma", "v_smfma"))


def _functions(asm: str):
    """(name, instructions) of every function of an assembly file, with the edges of its control flow."""
    name, body, labels, in_asm = None, [], {}, False

    def finish():
        target = None
        for i, ins in enumerate(body):
            for m in re.findall(r"\.LBB\w+", ins.line):
                target = m                               # (a long jump: s_getpc, s_add with the label, s_setpc)
            ends = ins.op in ("s_endpgm", "s_branch", "s_setpc_b64")
            after = [] if ends or i + 1 == len(body) else [i + 1]
            if ins.op.startswith(("s_branch", "s_cbranch", "s_setpc")):
                if labels.get(target, len(body)) < len(body):
                    after.append(labels[target])
            for j in after:
                ins.next.append(body[j])
                body[j].prev.append(ins)
        return name, body

    for raw in asm.splitlines():
        mark = raw.strip()
        if mark.startswith(";"):
            in_asm = "ASMSTART" in mark or (in_asm and "ASMEND" not in mark)
            continue
        line = re.sub(r"\s+", " ", raw.split(";")[0]).strip()
        m = re.match(r"([\w.$]+):", line)
        if m:
            if m.group(1).startswith("."):
                labels[m.group(1)] = len(body)
                continue
            if name and body:
                yield finish()
            name, body, labels = m.group(1), [], {}
        elif name and re.match(r"[a-z]+_", line):
            body.append(_Instr(line, in_asm))
    if name and body:
        yield finish()


def _walk(start: _Instr, edge: str, states: int):
    """Instructions fewer than `states` wait states away from `start`, with the distance in between."""
    best = {}
    todo = [(n, 0) for n in getattr(start, edge)]
    while todo:
        ins, dist = todo.pop()
        if dist >= states or best.get(ins, states) <= dist:
            continue
        best[ins] = dist
        todo.extend((n, dist + ins.states) for n in getattr(ins, edge))
    return best.items()


def hazards(asm: str) -> tuple[int, list[str]]:
    """The number of products written out as inline assembly, and what is too close to them."""
    count, found = 0, []
    for name, body in _functions(asm):
        products = [i for i in body if i.is_asm and i.is_product]
        count += len(products)
        if products:
            found += [f"{name}: scratch memory: {i.line}" for i in body if i.op.startswith("scratch_")]
        for p in products:
            result, operands = _regs(p.args[0]), _regs(",".join(p.args[1:]))
            for ins, dist in _walk(p, "prev", EXEC_WAIT):
                if not ins.op.startswith("v_") or not ins.args or ins.is_product:
                    continue                              # (products: the walk forward from them)
                if ins.op.startswith("v_cmpx") or ins.args[0] == "exec":
                    found.append(f"{name}: {ins.line} writes the lane mask {dist} wait states before {p.line}")
                written = _regs(ins.args[0]) | (_regs(ins.args[1]) if "swap" in ins.op else frozenset())
                if dist < OPERAND_WAIT and written & operands:
                    found.append(f"{name}: {ins.line} writes an operand {dist} wait states before {p.line}")
            for ins, dist in _walk(p, "next", RESULT_WAIT):
                if ins.is_product and ins.args[0] == p.args[0] == ins.args[3] and not _regs(",".join(ins.args[1:3])) & result:
                    continue
                if _regs(ins.line) & result:
                    found.append(f"{name}: {ins.line} touches the result {dist} wait states behind {p.line}")
        for ins in body:                                  # results of the compiler's own products in these operands
            if not products or not ins.is_product or ins.is_asm:
                continue
            result = _regs(ins.args[0])
            for p, dist in _walk(ins, "next", RESULT_WAIT):
                if p.is_asm and p.is_product and _regs(p.line) & result:
                    found.append(f"{name}: {p.line} uses a result {dist} wait states behind {ins.line}")
    return count, found
