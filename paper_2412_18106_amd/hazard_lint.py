"""Build-time check of the hand-issued instructions in the compiled kernels.

The attention kernel issues some MFMAs and LDS fragment reads as inline assembly
(see csrc/attn_kernels.hip for why).  The compiler schedules around them without
knowing what they are, so two things it normally guarantees have to be checked
on its output instead:

* the registers an inline-assembly MFMA writes are not read or written by any
  other kind of instruction (a register copy at a control-flow merge, a spill)
  before the wait states a vector-ALU access of an MFMA result needs have passed;
* the registers an inline-assembly ``ds_read`` writes are not touched before an
  ``s_waitcnt lgkmcnt`` has been issued;
* the registers an inline-assembly MFMA reads were not written by a vector-ALU
  instruction of the compiler's (a rematerialised constant, a copy) in the few
  wait states before it: the compiler pads that case for MFMAs it knows about.

* a scalar instruction in an inline-assembly statement that writes the SCC flag does not stand
  between a compare of the compiler's and the branch or select that reads it (the statement
  forgot to name "scc" among what it clobbers; met as a loop that never ended and then read
  out of bounds);

Everything the check reports is a real hazard of the path it names.  Backwards (operands of an MFMA) and
for the SCC flag it walks the assembly text straight through the basic block of the instruction.  Forwards (results
of MFMAs and of LDS reads) it does the same by default; with ``follow_branches``, as the build calls it, it goes on
through labels and barriers and takes both sides of every branch until the wait is over, since a copy where
control flow merges may stand behind a taken branch.
"""
from __future__ import annotations

import re

MFMA_WAIT_STATES = 12        # what the compiler pads between a 32x32x16 bf16 MFMA and a vector-ALU use of its result

VALU_TO_MFMA_WAIT_STATES = 4  # vector-ALU write of a register -> MFMA reading it

# scalar instructions that write SCC / that read it
_SCC_WRITERS = re.compile(r"^s_(add|sub|addc|subb|addk|and|or|xor|nand|nor|xnor|andn2|orn2|lshl|lshr|ashr|bfe|min|max|abs|"
                          r"absdiff|not|cmp|cmpk|bcnt0|bcnt1|wqm|quadmask|lshl[1-4]_add)_")
_SCC_READERS = re.compile(r"^s_(cbranch_scc[01]|cselect_b32|cselect_b64|addc_u32|subb_u32|cmov_b32|cmov_b64)\b")

_reg = re.compile(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b")
_AGPR = 1000                 # accumulation registers are numbered from here


def _regs(text):
    out = set()
    for m in _reg.finditer(text):
        if m.group(1) is not None:
            base = _AGPR if m.group(1) == "a" else 0
            out.update(range(base + int(m.group(2)), base + int(m.group(3)) + 1))
        else:
            base = _AGPR if m.group(4) == "a" else 0
            out.add(base + int(m.group(5)))
    return out


def _operands(line):
    line = line.split(";")[0].strip()
    parts = line.split(None, 1)
    if len(parts) < 2:
        return parts[0] if parts else "", [], ""
    ops = [o.strip() for o in parts[1].split(",")]
    return parts[0], ops, parts[1]


_LABEL = re.compile(r"^([.\w$]+):")
_CONTROL = ("s_cbranch", "s_branch", "s_endpgm", "s_setpc", "s_swappc")
# the address of a far jump: s_getpc_b64, two additions of the distance to the label, s_setpc_b64
_FAR = re.compile(r"\((\.L\w+)-")


def _next_lines(lines, labels, j, t):
    """Lines that may follow the control-flow instruction t on line j."""
    op = t.split()[0]
    if op == "s_endpgm":
        return []
    if op == "s_setpc_b64":
        far = next((m.group(1) for k in range(j - 1, max(j - 8, -1), -1) for m in [_FAR.search(lines[k])] if m), None)
        if far not in labels:
            raise ValueError(f"line {j + 1}: '{t}' jumps to an address this check cannot tell")
        return [labels[far]]
    target = t.split()[1] if op.startswith(("s_branch", "s_cbranch")) else None
    if target not in labels:
        raise ValueError(f"line {j + 1}: '{t}' goes to a place this check cannot tell")
    return [labels[target]] if op == "s_branch" else [j + 1, labels[target]]


def _walk(lines, labels, start, limit):
    """Yields (line, text, wait states passed) of the instructions that follow line start, until limit wait states have
    passed on a path; a true value sent back ends the path there.  labels: None stays in the basic block."""
    paths, least = [(start + 1, 0)], {}
    while paths:
        j, waited = paths.pop()
        while j < len(lines) and waited < limit:
            t = lines[j].strip()
            if not t or t.startswith(";") or (labels is not None and not t.startswith("s_") and (_LABEL.match(t) or t.startswith("."))):
                j += 1
                continue
            if labels is None and (t.endswith(":") or t.startswith(".")):
                break
            if least.get(j, limit) <= waited:
                break                     # this line has been reached with as little waiting before
            least[j] = waited
            if t.startswith(_CONTROL):
                if labels is not None:
                    paths += [(k, waited + 1) for k in _next_lines(lines, labels, j, t)]
                break
            if (yield j, t, waited):
                break
            op = t.split()[0]
            waited += int(t.split()[1]) + 1 if op == "s_nop" else 1
            j += 1


def _follow(lines, labels, start, limit, ends):
    """Line, text and wait states of the first instruction of a path behind line start for which ends says "hit"; "safe" ends
    a path without one."""
    walk = _walk(lines, labels, start, limit)
    try:
        j, t, waited = next(walk)
        while True:
            verdict = ends(t)
            if verdict == "hit":
                return j, t, waited
            j, t, waited = walk.send(verdict == "safe")
    except StopIteration:
        return None


def lint(asm_text, follow_branches=False):
    """Returns a list of (line number, message) for the hazards found in an AMDGPU assembly listing."""
    lines = asm_text.splitlines()
    labels = {m.group(1): i for i, line in enumerate(lines) for m in [_LABEL.match(line.strip())] if m} if follow_branches else None
    in_asm = False
    problems = []
    for i, raw in enumerate(lines):
        s = raw.strip()
        if s.startswith(";;#ASMSTART"):
            in_asm = True
            continue
        if s.startswith(";;#ASMEND"):
            in_asm = False
            continue
        if not in_asm:
            continue
        op, ops, _rest = _operands(s)
        if _SCC_WRITERS.match(op):
            depth = 1
            for j in range(i + 1, len(lines)):
                t = lines[j].strip()
                if t.startswith(";;#ASMEND"):
                    depth -= 1
                    continue
                if t.startswith(";;#ASMSTART"):
                    depth += 1
                    continue
                if not t or t.startswith(";") or depth > 0:
                    continue
                if t.endswith(":") or t.startswith(".") or t.startswith("s_branch") or t.startswith("s_endpgm"):
                    break
                o2 = t.split()[0]
                if _SCC_READERS.match(o2):
                    problems.append((j + 1, f"'{t}' reads the SCC flag that the inline-assembly '{s}' at line {i + 1} "
                                            "wrote (the statement does not declare \"scc\" as clobbered)"))
                    break
                if _SCC_WRITERS.match(o2):
                    break
        if op.startswith("v_mfma"):
            src = _regs(",".join(ops[1:]))
            waited = 0
            asm_depth = 1            # walking up: inside this MFMA's own statement first
            for j in range(i - 1, -1, -1):
                t = lines[j].strip()
                if t.startswith(";;#ASMEND"):
                    asm_depth += 1
                    continue
                if t.startswith(";;#ASMSTART"):
                    asm_depth -= 1
                    continue
                if not t or t.startswith(";"):
                    continue
                if t.endswith(":") or t.startswith("."):
                    break
                o2, ops2, rest2 = _operands(t)
                if o2 == "s_nop":
                    waited += int(ops2[0]) + 1
                else:
                    # asm_depth is 0 on the compiler's own instructions, 1 inside an inline-assembly statement
                    if asm_depth == 0 and o2.startswith("v_") and not o2.startswith("v_mfma") and ops2 \
                            and _regs(ops2[0]) & src:
                        problems.append((i + 1, f"hand-issued MFMA reads a register that '{t}' (line {j + 1}) wrote "
                                                f"{waited} wait states earlier (needs {VALU_TO_MFMA_WAIT_STATES})"))
                        break
                    waited += 1
                if waited >= VALU_TO_MFMA_WAIT_STATES:
                    break
            dst = _regs(ops[0])

            def ends(t):
                o2, ops2, rest2 = _operands(t)
                if o2 == "s_barrier" and not follow_branches:
                    return "safe"
                # (the matrix pipe orders MFMAs among themselves)
                return "hit" if not o2.startswith("v_mfma") and o2 != "s_nop" and _regs(rest2) & dst else None
            found = _follow(lines, labels, i, MFMA_WAIT_STATES, ends)
            if found:
                j, t, waited = found
                problems.append((j + 1, f"'{t}' touches the result of the hand-issued MFMA at line {i + 1} "
                                        f"after {waited} wait states (needs {MFMA_WAIT_STATES})"))
        elif op.startswith("ds_read"):
            dst = _regs(ops[0])

            def ends(t):
                o2, ops2, rest2 = _operands(t)
                if o2 == "s_waitcnt" and "lgkmcnt" in rest2:
                    return "safe"
                return "hit" if _regs(rest2) & dst else None
            found = _follow(lines, labels, i, 1 << 30, ends)
            if found:
                problems.append((found[0] + 1, f"'{found[1]}' touches the destination of the hand-issued LDS read at line {i + 1} "
                                               "before any s_waitcnt lgkmcnt"))
    return problems
