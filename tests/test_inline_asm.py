"""Inline assembly of the kernels: a statement that writes m0 says so.  The compiler does not look into the text, and would go on
using what it believes m0 to hold (the LDS base of its own loads into LDS, the index of a register move)."""
import glob
import os
import re

from paper_2601_03067_amd import build as kbuild

# the register as an instruction's first operand
WRITES_M0 = re.compile(r"(?:^|[\"\s;])(?!s_cmp|s_bitcmp)[sv]_\w+\s+m0\b")


def statements(text):
    """The operands of every asm statement, parentheses matched and string literals skipped over"""
    for m in re.finditer(r"\basm\b\s*(?:volatile|goto|\s)*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            ch = text[i]
            if ch == "\\":
                i += 1
            elif ch == '"':
                quoted = not quoted
            elif not quoted:
                depth += (ch == "(") - (ch == ")")
            i += 1
        yield text[m.end():i - 1]


def unnamed(text):
    return [s for s in statements(text) if WRITES_M0.search(s.replace("\\n", " ").replace("\\t", " ")) and '"m0"' not in s.rsplit(":", 1)[-1]]


def test_writes_to_m0_are_named_as_clobbers():
    n = 0
    for path in sorted(glob.glob(os.path.join(kbuild.CSRC, "*.hip")) + glob.glob(os.path.join(kbuild.CSRC, "*.h"))):
        with open(path) as f:
            text = f.read()
        n += sum(1 for _ in statements(text))
        assert not unnamed(text), path
    assert n > 20
    assert unnamed('asm volatile("s_mov_b32 m0, %0\\n\\tv_nop (x)" ::"s"(a) : "memory");')          # the check sees one
