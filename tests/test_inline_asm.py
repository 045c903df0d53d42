"""Wait states inside inline assembly.

gfx950 needs two wait states between a vector instruction that writes a scalar
register (a compare's or an add's condition, a lane read) and a vector
instruction that reads it.  The compiler inserts them in its own code; inside
an asm block the source has to hold them.  Every asm block of the kernels is
checked: each instruction counts one wait state, s_nop N counts N + 1.
"""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_04676_amd", "csrc")
SCALAR = re.compile(r"\b(?:vcc(?:_lo|_hi)?|s\d+|s\[\d+:\d+\])(?![\w:])")
NEEDED = 2


def asm_blocks(text):
    """The instructions of every asm statement, one list per statement."""
    for m in re.finditer(r'\basm\s+(?:volatile\s*)?\(\s*((?:"(?:[^"\\]|\\.)*"\s*)+)', text):
        body = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', m.group(1)))
        yield [i.strip() for i in re.split(r"\\n|;", body.replace("\\t", " ")) if i.strip()]


def short_waits(instructions):
    """(writer, reader) pairs of vector instructions too close to each other."""
    bad, writes = [], []                       # writes: (register, wait states since, instruction)
    for ins in instructions:
        op, _, rest = ins.partition(" ")
        args = [a.strip() for a in rest.split(",")] if rest else []
        if op.startswith("v_"):
            # operands written come first: the result, and an add's carry out
            dst = args[:2] if "_co_" in op else args[:1]
            src = " ".join(args[len(dst):])
            reads = set(SCALAR.findall(src))
            bad += [(w, ins) for reg, since, w in writes if reg in reads and since < NEEDED]
            writes = [(r, s + 1, w) for r, s, w in writes]
            writes += [(r, 0, ins) for d in dst for r in SCALAR.findall(d)]
        else:
            step = int(args[0], 0) + 1 if op == "s_nop" else 1
            writes = [(r, s + step, w) for r, s, w in writes]
    return bad


@pytest.mark.parametrize("instructions,ok", [
    (["v_cmp_ne_u32_e32 vcc, 0, %1", "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"], False),
    (["v_cmp_ne_u32_e32 vcc, 0, %1", "s_nop 0", "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"], False),
    (["v_cmp_ne_u32_e32 vcc, 0, %1", "s_nop 1", "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"], True),
    (["v_cmp_ne_u32_e64 s[4:5], 0, %1", "v_cndmask_b32_e64 %0, 0, 1, s[4:5]"], False),
    (["v_min_u32_e32 %1, 1, %2", "v_lshl_or_b32 %0, %0, 1, %1"], True),
])
def test_the_check_itself(instructions, ok):
    assert (not short_waits(instructions)) == ok


@pytest.mark.parametrize("name", sorted(f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp", ".h"))))
def test_asm_blocks_hold_their_wait_states(name):
    with open(os.path.join(CSRC, name)) as f:
        text = f.read()
    blocks = list(asm_blocks(text))
    assert len(blocks) == len(re.findall(r"\basm\s+volatile\s*\(|\basm\s*\(", text))
    for block in blocks:
        assert not short_waits(block), block
