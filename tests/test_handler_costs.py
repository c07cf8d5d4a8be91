"""HANDLER_VALU of bench.py against the interpreter's macros: the vector
instructions per case of each operator's fast handler in interp_gfx950.h, range
tests left out."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MACROS = {5: ("GP_DIV",), 6: ("GP_SIN", "GP_SINBODY"), 7: ("GP_COS", "GP_SINBODY"), 8: ("GP_EXP",), 9: ("GP_LOG",)}


def _asm():
    text = open(os.path.join(ROOT, "paper_2607_06731_amd", "csrc", "interp_gfx950.h")).read()
    return text[text.index('R"(') + 3:text.index(')");')]


def _per_case(asm, macro):
    """Vector instructions in a macro's loops over the cases."""
    body = re.search(r"^\.macro %s\b[^\n]*\n(.*?)^\.endm" % macro, asm, re.S | re.M).group(1)
    loops = re.findall(r"\.irp j,0,1,2,3\n(.*?)\.endr", body, re.S)
    rest = re.sub(r"\.irp j,0,1,2,3\n.*?\.endr", "", body, flags=re.S)
    assert not re.search(r"^\s+v_", rest, re.M), macro
    return sum(len(re.findall(r"^\s+v_", b, re.M)) for b in loops)


def test_costs_are_the_macros():
    sys.path.insert(0, ROOT)
    import bench
    asm = _asm()
    for op, names in MACROS.items():
        assert bench.HANDLER_VALU[op] == sum(_per_case(asm, n) for n in names), op
    assert bench.HANDLER_VALU[:5] == (0, 0, 1, 1, 1)
    # a square root and a magnitude: one instruction per case in their handlers
    for off, op in ((3200, 10), (3296, 11)):
        part = asm[asm.index(", %d, \\last" % off):]
        part = part[:part.index("GP_NEXT")]
        loop = re.search(r"\.irp j,0,1,2,3\n(.*?)\.endr", part, re.S).group(1)
        assert len(re.findall(r"^\s+v_", loop, re.M)) == bench.HANDLER_VALU[op]
