"""No instruction touches a register that a load has yet to fill.

The compiler takes the outputs of inline assembly as written when the statement ends, so for a load that stands in a statement of its
own it neither waits nor keeps the registers free until the data is there.  The compiled kernels are walked here along every path:
a destination is pending from its load until a counter wait that covers it, and nothing may read or write it in between.
"""
import os
import re
import subprocess

import pytest

from paper_2502_14477_amd import build

LISTED = re.compile(r"([va])(?:(\d+)|\[(\d+):(\d+)\])(?![\w\[])")
COUNTER_MAX = 64


def registers(text):
    """{'v12', 'a3', ...} of one operand or a list of them."""
    found = set()
    for kind, one, lo, hi in LISTED.findall(text):
        found |= {kind + str(i) for i in (range(int(lo), int(hi) + 1) if lo else (int(one),))}
    return found


def waits(operands):
    """(vmcnt, lgkmcnt) of an s_waitcnt, COUNTER_MAX where it does not wait for one."""
    if re.fullmatch(r"(0x[0-9a-f]+|\d+)", operands.strip()):
        code = int(operands, 0)
        vm, lgkm = (code & 15) | (code >> 10 & 48), code >> 8 & 15
        return (COUNTER_MAX if vm == 63 else vm), (COUNTER_MAX if lgkm == 15 else lgkm)
    at = {name: int(n) for name, n in re.findall(r"(vmcnt|lgkmcnt)\((\d+)\)", operands)}
    return at.get("vmcnt", COUNTER_MAX), at.get("lgkmcnt", COUNTER_MAX)


def counter_of(op):
    """Which counter an instruction raises; LDS operations complete in order, vector memory operations too."""
    if op.startswith("ds_"):
        return "lgkm"
    return "vm" if op.startswith(("global_", "buffer_", "scratch_", "flat_")) and not op.startswith(("buffer_wbl2", "buffer_inv")) else None


def loaded(op, operands):
    """The registers a load fills."""
    if "_lds" in op or op.startswith(("ds_write", "ds_max_u32", "ds_add_u32", "ds_or_b32")) or "store" in op:
        return set()
    if op.startswith("ds_") or "_load_" in op or ("_atomic_" in op and re.search(r"\b(sc0|glc)\b", operands)):
        return registers(operands.split(",")[0])
    return set()


def functions(listing):
    """{name: [(label, ...) or (op, operands), ...]} of a compiler's assembly listing."""
    found, name = {}, None
    for line in listing.splitlines():
        line = line.split(";")[0].split("//")[0].strip()
        if re.fullmatch(r"_Z\w+:", line):
            name = line[:-1]
            found[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and re.fullmatch(r"\.L\w+:", line):
            found[name].append((line[:-1],))
        elif name and line and not line.startswith("."):
            op, _, operands = line.partition(" ")
            found[name].append((op.strip(), operands.strip()))
    return found


def touched_while_pending(code):
    """[(index, instruction, registers)] of one function."""
    labels = {c[0]: i for i, c in enumerate(code) if len(c) == 1}
    starts = sorted({0} | set(labels.values()) | {i + 1 for i, c in enumerate(code) if c[0].startswith(("s_branch", "s_cbranch", "s_endpgm"))})
    end_of = dict(zip(starts, starts[1:] + [len(code)]))
    entry = {0: {}}                                  # block -> {register: (counter, operations issued behind it)}, the fewest over all paths
    todo, hits = [0], {}
    while todo:
        at = todo.pop()
        state, following = dict(entry[at]), [end_of[at]]
        for i in range(at, end_of[at]):
            if len(code[i]) == 1:
                continue
            op, operands = code[i]
            if op == "s_waitcnt":
                left = dict(zip(("vm", "lgkm"), waits(operands)))
                state = {r: p for r, p in state.items() if p[1] < left[p[0]]}
                continue
            assert not op.startswith(("s_setpc", "s_swappc", "s_call")), "a call"
            counter = counter_of(op)
            touched = {r for r in registers(operands) if r in state}
            if loaded(op, operands):                  # loads of one counter arrive in order: the later one stays
                sources = registers(operands.partition(",")[2])
                touched = {r for r in touched if r in sources or state[r][0] != counter}
            if touched:
                hits[i] = (i, op + " " + operands, touched)
            if counter:
                state = {r: (c, n + 1 if c == counter else n) for r, (c, n) in state.items() if n < COUNTER_MAX}
                state.update({r: (counter, 0) for r in loaded(op, operands)})
            if op.startswith(("s_branch", "s_cbranch")):
                following = [labels[operands]] + ([] if op == "s_branch" else [i + 1])
            elif op == "s_endpgm":
                following = []
        for to in following:
            if to >= len(code):
                continue
            known = entry.get(to)
            merged = dict(known or {})
            for r, p in state.items():
                if r not in merged or p[1] < merged[r][1]:
                    merged[r] = p
            if known is None or merged != known:
                entry[to] = merged
                todo.append(to)
    return [hits[i] for i in sorted(hits)]


def listing_of(source):
    flags = build.FLAGS + build.EXTRA_FLAGS.get(source, [])
    cmd = [build._hipcc(), *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", "-"]
    return subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.DEVNULL, text=True).stdout


def test_the_walk_sees_what_it_looks_for():
    code = """_Zk:
	s_cbranch_scc1 .LBB0_2
	ds_read_b128 v[4:7], v0
	ds_read_b128 v[8:11], v0
.LBB0_2:
	s_waitcnt lgkmcnt(1)
	v_add_f32_e32 v4, v4, v5
	%s
	v_mov_b32_e32 v9, 0
	s_endpgm
.Lfunc_end0:
"""
    walk = lambda text: touched_while_pending(functions(code % text)["_Zk"])
    assert [h[1:] for h in walk("s_nop 0")] == [("v_mov_b32_e32 v9, 0", {"v9"})]
    assert walk("s_waitcnt lgkmcnt(0)") == [] and walk("s_waitcnt 0xc07f") == [] and walk("ds_write_b32 v0, v1\n\ts_waitcnt lgkmcnt(1)") == []
    assert len(walk("global_load_dword v9, v1, s[0:1]")) == 2 and len(walk("s_waitcnt vmcnt(0)")) == 1


@pytest.mark.parametrize("source", ["score.hip", "attend_split.hip", "compress.hip"])        # those with loads in inline assembly
def test_no_register_is_touched_while_a_load_into_it_is_pending(source):
    found = functions(listing_of(source))
    assert found
    hits = {name: touched_while_pending(code) for name, code in found.items()}
    assert not any(hits.values()), {name: h[:8] for name, h in hits.items() if h}
