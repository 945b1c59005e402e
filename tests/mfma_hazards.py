"""Wait states around the MFMA instructions of a compiled kernel.

The bounded attention kernel issues its MFMAs from inline assembly, which the
compiler's hazard recogniser does not see: the kernel itself has to keep an
MFMA's result registers away from every other reader or writer until the MFMA
is through, and freshly written registers away from an MFMA that reads them.
``violations`` reads the assembly of a kernel and lists where that fails.

An instruction counts one wait state, ``s_nop n`` counts n + 1 (an MFMA that
waits for the matrix unit takes longer: the count is a lower bound).  At a
label the shortest distance over all ways to reach it counts.
"""
import re

RESULT_WAIT = 19    # MFMA result -> any instruction but an MFMA that accumulates on the same registers
OPERAND_WAIT = 2    # VALU write -> MFMA operand


def functions(asm, pattern):
    """{name: [(line, instruction or label)]} of the kernels whose mangled name matches pattern."""
    out, name = {}, None
    for n, line in enumerate(asm.splitlines(), 1):
        text = line.split(";")[0].strip()
        m = re.match(r"(_Z\w+):", text)
        if m:
            name = m.group(1) if re.search(pattern, m.group(1)) else None
            if name:
                out[name] = []
        elif text.startswith(".Lfunc_end"):
            name = None
        elif name and text and (not text.startswith(".") or text.endswith(":")):
            out[name].append((n, text))
    return out


def _regs(operand):
    m = re.fullmatch(r"[-|]*([va])(?:(\d+)|\[(\d+):(\d+)\])\|?", operand)
    if not m:
        return frozenset()
    lo, hi = (m.group(2), m.group(2)) if m.group(2) else (m.group(3), m.group(4))
    return frozenset((m.group(1), r) for r in range(int(lo), int(hi) + 1))


def _parse(text):
    op, _, rest = text.partition(" ")
    return op, [o.split(" ")[0] for o in re.split(r",\s*", rest.strip())] if rest else []


def violations(body):
    """[(line, text)] of the instructions of one kernel that come too early after an MFMA or a register write."""
    blocks, label_of = [[]], {}
    for n, text in body:
        if text.endswith(":"):
            if blocks[-1]:
                blocks.append([])
            label_of[text[:-1]] = len(blocks) - 1
        else:
            blocks[-1].append((n, text))
            if text.startswith(("s_branch", "s_cbranch", "s_endpgm")):
                blocks.append([])
    found = {}

    def run(i, state):
        # state: register -> [wait states since an MFMA wrote it, its whole result; since a VALU instruction did]
        mfma, valu = {r: list(v) for r, v in state[0].items()}, dict(state[1])
        for n, text in blocks[i]:
            op, args = _parse(text)
            regs = [_regs(a) for a in args]
            touched = frozenset().union(*regs) if regs else frozenset()
            if op.startswith("v_mfma"):
                dst, src_c = regs[0], regs[3]
                early = [r for r in touched if r in mfma and not (dst == mfma[r][1] and r in dst and src_c in (dst, frozenset()))]
                early += [r for s in regs[1:] for r in s if valu.get(r, 99) < OPERAND_WAIT]
            else:
                early = [r for r in touched if r in mfma]
            if early:
                found[n] = text
            steps = int(args[0]) + 1 if op == "s_nop" else 1
            for r in [r for r, v in mfma.items() if v[0] + steps >= RESULT_WAIT]:
                del mfma[r]
            for v in mfma.values():
                v[0] += steps
            valu = {r: a + steps for r, a in valu.items() if a + steps < OPERAND_WAIT}
            if op.startswith("v_mfma"):
                for r in regs[0]:
                    mfma[r] = [0, regs[0]]
            elif op.startswith("v_") and regs:
                for r in regs[0] | (regs[1] if "swap" in op else frozenset()):
                    valu[r] = 0
        return mfma, valu

    # shortest distances at every block entry
    entry = {0: ({}, {})}
    work = [0]
    while work:
        i = work.pop()
        mfma, valu = run(i, entry[i])
        last = blocks[i][-1][1] if blocks[i] else ""
        succ = [] if last.startswith(("s_branch", "s_endpgm")) else [i + 1]
        if last.startswith(("s_branch", "s_cbranch")):
            succ.append(label_of[last.split()[-1]])
        for s in succ:
            if s >= len(blocks):
                continue
            new = s not in entry
            em, ev = entry.setdefault(s, ({}, {}))
            for r, v in mfma.items():
                if r not in em or v[0] < em[r][0]:
                    em[r] = list(v)
                    new = True
            for r, a in valu.items():
                if a < ev.get(r, 99):
                    ev[r] = a
                    new = True
            if new and s not in work:
                work.append(s)
    return sorted(found.items())
