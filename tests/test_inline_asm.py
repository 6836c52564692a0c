"""Inline assembly tells the compiler what it changes: a statement that writes
m0 or scc names it among its clobbers."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_20791_amd", "csrc")


def _asm_statements():
    for f in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, f)).read()
        for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\((.*?)\);", text, re.S):
            yield pytest.param(m.group(1), id="%s:%d" % (f, text.count("\n", 0, m.start()) + 1))


@pytest.mark.parametrize("stmt", _asm_statements())
def test_written_registers_are_clobbers(stmt):
    template = re.match(r'\s*"(?:[^"\\]|\\.)*"', stmt).group(0)
    last = re.search(r':\s*((?:"\w+"\s*,?\s*)+)$', stmt)  # clobbers are bare names, operands have values
    clobbers = last.group(1) if last else ""
    if re.search(r"\bm0\s*,", template):
        assert '"m0"' in clobbers
    if re.search(r"\bs_(add|sub|addc|subb|and|or|xor|lsh[lr]|cmp)\w*\b", template):
        assert '"scc"' in clobbers
