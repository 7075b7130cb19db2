"""Checks of the device sources and of what the compiler made of them, without
a GPU."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_14681_amd", "csrc")


def asm_statements(text):
    """The text of every asm(...) statement, parentheses matched outside string literals."""
    for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(", text):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = text[i]
            if c == "\\" and quoted:
                i += 1
            elif c == '"':
                quoted = not quoted
            elif not quoted:
                depth += (c == "(") - (c == ")")
            i += 1
        yield text[m.start():i]


def test_inline_asm_names_the_m0_it_writes():
    """An asm statement that writes M0 lists it as clobbered: the compiler
    may keep a value of its own there (indexed moves, LDS-DMA builtins,
    messages)."""
    writers = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            for s in asm_statements(f.read()):
                if re.search(r"\bm0\s*,", s):
                    writers.append((os.path.basename(path), s))
    assert writers
    for path, s in writers:
        assert re.search(r':\s*(?:"\w+"\s*,\s*)*"m0"', s), (path, s)
