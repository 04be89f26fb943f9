"""Device code holds no instruction as inline assembly.  The compiler puts the
waits that matrix and dot products need around the instructions it knows; what
an inline instruction reads and writes is hidden from it, so one that
overwrites an operand of a product still running, or reads its result too
early, gets no wait.  (Empty statements, which only tie a value to a register,
emit nothing and are fine.)"""
import os
import re

import paper_1710_08591_amd.build as b


def test_no_inline_instructions():
    found = []
    for name in sorted(os.listdir(b.CSRC)):
        with open(os.path.join(b.CSRC, name)) as f:
            text = re.sub(r"//[^\n]*", "", f.read())
        for m in re.finditer(r'\basm\b\s*(?:volatile|__volatile__)?\s*\(\s*"((?:[^"\\]|\\.)*)"', text):
            if m.group(1).strip():
                found.append((name, m.group(1)))
        assert "__asm" not in text, name
    assert not found
