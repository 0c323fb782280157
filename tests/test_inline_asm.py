"""What the kernel sources have to tell the compiler beyond the language: registers that inline assembly changes, and the
order of LDS accesses that different lanes of a wave make to the same place."""
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


def test_areas_exchanged_within_a_wave_are_ordered_on_both_sides():
    """Both fp32 epilogues read the partner's sums, write the finished tile over them and read it in row order."""
    for name in ("gemm_mfma.h", "gemm_rows.h"):
        text = open(os.path.join(CSRC, name)).read()
        at = text.index("float4* t = ")
        write, read = re.search(r"\bt\[lm \* \d", text[at:]).start(), re.search(r"= t\[r \* \d", text[at:]).start()
        assert "wave_lds_order();" in text[at:at + write] and "wave_lds_order();" in text[at + write:at + read], name
