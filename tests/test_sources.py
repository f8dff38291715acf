"""Rules of the kernel sources that a compiler does not check."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_14477_amd", "csrc")


def asm_statements():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        for m in re.finditer(r"\basm\s+volatile\s*\((.*?)\)\s*;", open(path).read(), re.S):
            yield os.path.basename(path), m.group(1)


def test_inline_assembly_that_writes_m0_says_so():
    """m0 holds the LDS address of the compiler's own loads into LDS too: it has to know when a statement changes it."""
    writers = [(f, s) for f, s in asm_statements() if re.search(r"\bs_mov_b32 m0\b", s)]
    assert writers
    for f, s in writers:
        clobbers = s.rsplit(":", 1)[-1]
        assert '"m0"' in clobbers, (f, s)
