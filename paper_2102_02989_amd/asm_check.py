"""Check of the generated gfx950 assembly for per-lane instructions in front of
an exec restore.

Where a divergent region ends, the block in which its lanes meet again opens with
the restore of the exec mask (s_or_b64 exec, exec, ...).  Close to the register
limit the compiler of ROCm 7.2 can put the copy of a spilled register (to an
accumulation register or to scratch memory) in front of that restore: it does
so when a scalar copy already stands there.  The copy then runs with the lanes that
left the region switched off, and their value, an address for instance, is lost:
wrong results or an access out of bounds, without a word from the compiler.

Two kinds of blocks are certain to be such meeting points: the target of an
s_cbranch_execz (the edge on which a region with no active lane is skipped)
and the block behind the s_cbranch_execnz that closes a divergent loop.  In
neither may an instruction that works per lane precede the restore.  (v_readlane,
v_readfirstlane and v_writelane move scalars and do not depend on the mask.)"""
from __future__ import annotations

import re

_PER_LANE = re.compile(r"(v_(?!readlane|readfirstlane|writelane|nop)|scratch_|ds_|global_|buffer_|flat_)")
_LABEL = re.compile(r"(\.LBB\w+):")
_KERNEL = re.compile(r"([A-Za-z_]\w*):")


def check(text: str) -> tuple[int, list[tuple[str, int, str]]]:
    """(exec restores looked at, findings); a finding is (function, line of the
    restore, the per-lane instruction in front of it)."""
    lines = text.splitlines()
    skip = {ln.split()[1] for ln in lines if ln.startswith("\ts_cbranch_execz")}
    func, found, n = "", [], 0
    meet, ops, written, prev = False, [], set(), ""
    for num, line in enumerate(lines, 1):
        label = _LABEL.match(line)
        if label or line.startswith("; %bb"):
            meet = (label is not None and label.group(1) in skip) or prev.startswith("s_cbranch_execnz")
            ops, written = [], set()
            continue
        if not line.startswith("\t"):
            if _KERNEL.match(line):
                func, meet, prev = _KERNEL.match(line).group(1), False, ""
            continue
        ins = line.split(";")[0].strip()
        if not ins or ins.startswith("."):
            continue
        op, _, rest = ins.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        # (a saved mask moved back whole; one computed in the block narrows the mask)
        restore = args[0] == "exec" and (op == "s_or_b64" or (op == "s_mov_b64" and args[1] not in written))
        if meet and restore:
            n += 1
            if ops:
                found.append((func, num, ops[0]))
        if args[0] == "exec" or "saveexec" in op or op.startswith(("s_cbranch", "s_branch", "v_cmpx")):
            meet = False
        elif meet:
            written.add(args[0])
            if _PER_LANE.match(op):
                ops.append(ins)
        prev = ins
    return n, found
