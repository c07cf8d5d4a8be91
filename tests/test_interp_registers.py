"""The registers that the interpreter's handlers write
(paper_2607_06731_amd/csrc/interp_gfx950.h) against the operand and clobber
lists of the statement that enters them (GP_THREAD_ASM in gpeval.hip): every
explicit destination and every register that an instruction writes by itself is
declared, so the compiler keeps nothing there."""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2607_06731_amd", "csrc")

# written without being named: opcode pattern -> register
IMPLICIT = [(r"s_(add|addc|sub|subb|and|or|lshl|lshr|bfe|cmp)\w*", "scc"),
            (r"v_cmp\w*_e32", "vcc"), (r"v_div_fmas\w*", None),
            (r"s_set_gpr_idx_on", "m0"), (r"s_(mov|add)\w* m0", "m0")]


def _declared():
    text = open(os.path.join(CSRC, "gpeval.hip")).read()
    m = re.search(r"#define GP_THREAD_ASM\(.*?\n\n", text, re.S)
    body = m.group(0)
    regs = set()
    for a in re.findall(r"\{([^}]+)\}", body) + re.findall(r'"([a-z]+\d*)"', body):
        r = re.fullmatch(r"([vs])\[(\d+):(\d+)\]", a)
        if r:
            regs |= {r.group(1) + str(k) for k in range(int(r.group(2)), int(r.group(3)) + 1)}
        elif re.fullmatch(r"[vs]\d+|vcc|scc|m0|exec", a):
            regs.add(a)
    return regs


def _instructions():
    """(opcode, operands) of every instruction line of the macros."""
    text = open(os.path.join(CSRC, "interp_gfx950.h")).read()
    asm = text[text.index('R"(') + 3:text.index(')");')]
    for line in asm.splitlines():
        line = line.split("//")[0].strip()
        m = re.match(r"((?:v|s|ds)_\\?\w+(?:\\\(\))?\w*)\s*(.*)", line)
        if m:
            yield m.group(1), m.group(2)


def test_every_written_register_is_declared():
    regs = _declared()
    seen = 0
    for op, args in _instructions():
        for pat, reg in IMPLICIT:
            if reg and re.match(pat, op + " " + args):
                assert reg in regs, (op, args, reg)
        if op.startswith(("s_cbranch", "s_branch", "s_setpc", "s_waitcnt", "s_nop", "s_set_gpr_idx", "s_cmp")):
            continue
        dst = args.split(",")[0].strip()
        m = re.fullmatch(r"([vs])\[?(\d+)(?::(\d+))?\]?", dst)
        if m:                              # numbered registers (cells and temporaries by case: below)
            lo, hi = int(m.group(2)), int(m.group(3) or m.group(2))
            for k in range(lo, hi + 1):
                assert m.group(1) + str(k) in regs, (op, args)
            seen += 1
        if op.startswith("v_div_scale"):
            second = args.split(",")[1].strip()
            want = {"vcc"} if second == "vcc" else {"s96", "s97"}
            assert want <= regs
        if op.startswith("v_swap"):
            continue
    assert seen > 30
    # temporaries v4..v18 by case, cells v36..v67, compare masks s68..s75
    assert {"v%d" % k for k in range(4, 19)} <= regs
    assert {"v%d" % k for k in range(36, 68)} <= regs
    assert {"s%d" % k for k in range(68, 76)} <= regs


def test_the_index_mode_needs_m0():
    ops = [op for op, _ in _instructions()]
    assert ops.count("s_set_gpr_idx_on") == 4
    assert "m0" in _declared()
