"""Checks of the HIP sources that need no GPU: inline assembly states every register it writes."""
import glob
import os
import re

from tests.conftest import ROOT


def asm_statements(src):
    """The argument text of every asm statement of a source (string literals may hold parentheses)."""
    for m in re.finditer(r"\basm\s+volatile\s*\(", src):
        depth, i, quoted = 1, m.end(), False
        while depth:
            c = src[i]
            if quoted:
                i += c == "\\"
                quoted = c != '"'
            elif c == '"':
                quoted = True
            else:
                depth += (c == "(") - (c == ")")
            i += 1
        yield src[m.end():i - 1]


def test_asm_that_writes_m0_declares_it():
    found = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2608_11235_amd", "csrc", "*"))):
        with open(path) as f:
            for text in asm_statements(f.read()):
                strings = re.findall(r'"((?:[^"\\]|\\.)*)"', text)
                if re.search(r"\bs_mov_b32\s+m0\b", text):
                    found += 1
                    assert "m0" in strings, f"{os.path.basename(path)}: m0 not clobbered in asm({text})"
    assert found
