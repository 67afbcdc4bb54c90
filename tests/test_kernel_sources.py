"""Inline assembly in the HIP sources names every register that it writes besides its operands."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_24211_amd", "csrc")
# instructions that write one of these as their destination, or scc as a side effect
WRITES = {"m0": r"\bs_\w+ m0\b", "vcc": r"\b[sv]_\w+ vcc\b", "scc": r"\bs_(add|sub|and|or|xor|cmp|lshl|lshr)\w* "}


def _statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = open(path).read()
        for m in re.finditer(r"\basm\s*(?:volatile\s*)?\(", text):
            depth, end = 1, m.end()
            while depth:
                depth += {"(": 1, ")": -1}.get(text[end], 0)
                end += 1
            yield os.path.basename(path), text[m.end():end - 1]


def test_asm_names_what_it_clobbers():
    found = 0
    for name, body in _statements():
        code = re.match(r'\s*((?:"(?:[^"\\]|\\.)*"\s*)+)', body).group(1)
        clobbers = body.rsplit(":", 1)[1] if body.count(":") >= 3 else ""
        for register, pattern in WRITES.items():
            if re.search(pattern, code):
                found += 1
                assert f'"{register}"' in clobbers, (name, register, code)
    assert found >= 4      # both forms of the load to LDS write m0 and scc
