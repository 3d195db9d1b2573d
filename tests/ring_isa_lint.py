"""Static check of the ring prefill kernels' gfx950 assembly.

The unit loop of csrc/prefill_bf16_ring.hip issues its LDS reads (and one scalar load) as inline
assembly that the compiler does not track, and waits for them by count.  The compiler believes such a
value is there as soon as the instruction has been issued, so nothing but the kernel's own waits keeps
it from touching the destination registers too early: a copy, a spill, or -- once the value is dead in
its eyes -- a reuse of the registers for something else while the read is still in flight, which
then lands on top of the new contents.  This module replays every kernel's instruction stream with a
model of the LDS counter (operations of a wave complete in order; s_waitcnt lgkmcnt(N) returns when
at most N are outstanding; scalar loads return out of order and are only known to be back after
lgkmcnt(0)) and reports every instruction that reads or writes a register while a load into it may
still be in flight.  Both sides of every branch are followed, each with the state at the branch, until no
new state turns up: a wait counts on the paths that run it alone.
"""
from __future__ import annotations

import re
from typing import List, Tuple

_REG = re.compile(r"\b([vsa])(\d+)\b|\b([vsa])\[(\d+):(\d+)\]")


def _regs(text: str):
    out = set()
    for m in _REG.finditer(text):
        if m.group(1):
            out.add((m.group(1), int(m.group(2))))
        else:
            out.update((m.group(3), i) for i in range(int(m.group(4)), int(m.group(5)) + 1))
    return out


def kernels(asm_text: str):
    """Yields (name, [instruction lines]) for every kernel body in an assembly file."""
    name, body = None, []
    for line in asm_text.splitlines():
        m = re.match(r"^(_Z\w+):", line)
        if m:
            name, body = m.group(1), []
            continue
        if name is None:
            continue
        s = line.strip()
        if s.startswith(".Lfunc_end"):
            if any("s_endpgm" in b for b in body):
                yield name, body
            name = None
            continue
        if not s or s.startswith(";") and "ASM" not in s or s.startswith(".") and not s.startswith(".LBB"):
            continue
        body.append(s.split(";")[0].strip() if not s.startswith(";;#ASM") else s)


# Operations that a state remembers one by one; older ones are remembered together (waits ask for at most 15).
_REMEMBERED = 64


def _parse(ins: str):
    """(kind, argument, registers touched, registers loaded) of one instruction line."""
    if not ins or ins.startswith(";;#ASM") or ins.endswith(":"):
        return ("", None, frozenset(), frozenset())
    op, _, operands = ins.partition(" ")
    if op == "s_waitcnt":
        m = re.search(r"lgkmcnt\((\d+)\)", ins)
        return ("wait" if m else "", int(m.group(1)) if m else None, frozenset(), frozenset())
    touched = frozenset(_regs(operands))
    if op.startswith(("ds_read", "ds_load")):
        return ("lds", None, touched, frozenset(_regs(operands.split(",")[0])))
    if op.startswith(("ds_write", "ds_store")):
        return ("lds", None, touched, frozenset())
    if op.startswith(("s_load", "s_buffer_load")):
        return ("scalar", None, touched, frozenset(_regs(operands.split(",")[0])))
    if op == "s_endpgm":
        return ("end", None, touched, frozenset())
    if op == "s_branch" or op.startswith("s_cbranch"):
        return ("jump" if op == "s_branch" else "branch", ins.split()[-1], touched, frozenset())
    assert not op.startswith(("s_setpc", "s_swappc", "s_call")), "control flow that is not followed: " + ins
    return ("", None, touched, frozenset())


def lint(body: List[str]) -> List[Tuple[int, str, str]]:
    """Returns (line index, instruction, reason) for every hazard found in one kernel body, in order."""
    labels = {l[:-1]: i for i, l in enumerate(body) if l.startswith(".LBB") and l.endswith(":")}
    code = [_parse(ins) for ins in body]
    problems = {}
    start = (0, (), frozenset())  # line, LDS operations in flight (oldest first), scalar loads in flight
    seen, todo = {start}, [start]

    def go(state):
        if state not in seen:
            seen.add(state)
            todo.append(state)

    while todo:
        i, fifo, scalar = todo.pop()
        fifo, scalar = list(fifo), set(scalar)
        while i < len(body):
            kind, arg, touched, loaded = code[i]
            if touched:
                for dest in fifo + list(scalar):
                    if touched & dest:  # (a load into a register that another is in flight into is a hazard too)
                        problems[i] = (i, body[i], "touches %s while a load into it may be in flight" % sorted(touched & dest)[:4])
                        break
            if kind == "wait":
                del fifo[:max(0, len(fifo) - arg)]
                if arg == 0:
                    scalar.clear()
            elif kind == "lds":
                fifo.append(loaded)
                if len(fifo) > _REMEMBERED:
                    fifo[:2] = [fifo[0] | fifo[1]]
            elif kind == "scalar":
                scalar.add(loaded)
            elif kind == "end":
                break
            elif kind == "jump":
                go((labels[arg], tuple(fifo), frozenset(scalar)))
                break
            elif kind == "branch":
                go((labels[arg], tuple(fifo), frozenset(scalar)))
                go((i + 1, tuple(fifo), frozenset(scalar)))
                break
            i += 1
            if i < len(body) and body[i].endswith(":"):  # where paths meet
                go((i, tuple(fifo), frozenset(scalar)))
                break
    return [problems[i] for i in sorted(problems)]
