"""Inline assembly in the kernel sources tells the compiler every register it changes."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_04147_amd", "csrc")


def test_statements_that_write_m0_declare_it():
    seen = 0
    for path in glob.glob(os.path.join(CSRC, "*")):
        for text, rest in re.findall(r'asm volatile\(((?:\s*"(?:[^"\\]|\\.)*")+)([^;]*);', open(path).read()):
            if re.search(r"\bm0\s*,", text):                 # m0 as a destination operand
                seen += 1
                assert re.search(r':[^:]*"m0"[^:]*\)\s*$', rest), (os.path.basename(path), text)
    assert seen == 1
