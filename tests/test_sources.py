"""Rules of the kernel sources and of figures tied to them that a compiler does not check."""
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


def test_measured_traffic_is_tied_to_the_compiler_flags(monkeypatch):
    """A flag changes the code of every kernel as a change to its source does; where the tree lies does not."""
    import bench
    from paper_2502_14477_amd import build
    here = bench.csrc_tree_hash()
    at = build.FLAGS.index("-I") + 1
    monkeypatch.setattr(build, "FLAGS", build.FLAGS[:at] + ["/elsewhere/include"] + build.FLAGS[at + 1:])
    assert bench.csrc_tree_hash() == here
    monkeypatch.setattr(build, "FLAGS", ["-O2" if f == "-O3" else f for f in build.FLAGS])
    other = bench.csrc_tree_hash()
    assert other != here
    monkeypatch.setattr(build, "EXTRA_FLAGS", {})
    assert bench.csrc_tree_hash() not in (here, other)
