"""Static check of the compiled kernels: a vector-memory instruction may read a scalar register at the earliest five
wait states after a vector instruction (v_readfirstlane, v_readlane) wrote it.  The compiler keeps the distance for its
own loads but not for loads by inline asm, which then go out with the register's old value, such as another operand's
buffer descriptor."""
import os
import re

import pytest

from tests.test_store_hazard_scan import HIPCC, SOURCES, _assembly, _instructions

WAIT_STATES = 5
MEMORY = ("buffer_", "global_", "flat_", "scratch_")


def scan_scalar_reads(asm: str) -> list:
    """(function, writer, reader) of every pair that is too close, in program order."""
    insts, hits = _instructions(asm), []
    for i, (fn, s) in enumerate(insts):
        if not s.startswith(MEMORY):
            continue
        reads = {int(x) for x in re.findall(r"\bs(\d+)\b", s)}
        for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", s):
            reads |= set(range(int(a), int(b) + 1))
        waited = 0
        for fn2, s2 in reversed(insts[max(0, i - 2 * WAIT_STATES):i]):
            if fn2 != fn or waited >= WAIT_STATES:
                break
            op = s2.split()[0]
            if op == "s_branch":
                break  # what stands before it does not fall through to the load
            if op.startswith(("v_readfirstlane", "v_readlane")) and int(re.search(r"\bs(\d+)\b", s2).group(1)) in reads:
                hits.append((fn, s2, s))
            waited += int(s2.split()[1]) + 1 if op == "s_nop" else 1
    return hits


def test_scanner_finds_the_pattern():
    load = "\tbuffer_load_dwordx4 v7, s[4:7], 0 offen lds\n"
    near = "k:\n\tv_readfirstlane_b32 s6, v189\n\tv_readfirstlane_b32 s9, v189\n\ts_mov_b32 m0, s3\n\ts_nop 0\n"
    assert len(scan_scalar_reads(near + load)) == 1
    assert scan_scalar_reads(near + "\ts_nop 1\n" + load) == []
    assert scan_scalar_reads(near.replace("s6", "s8") + load) == []


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("src", SOURCES)
def test_no_load_reads_a_scalar_too_early(src):
    hits = scan_scalar_reads(_assembly(src))
    assert not hits, "\n".join(f"{fn}: [{a}] then [{b}]" for fn, a, b in hits[:10])


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_backward_products_keep_both_kinds_of_stores():
    # the compiler takes a non-temporal store and a plain one of the same value for the same and may join them into plain ones
    src = next(s for s in SOURCES if "lmhead" in str(s))
    kinds = {}
    for fn, inst in _instructions(_assembly(src)):
        if "k_lm_backward" in fn and inst.startswith("global_store_dword "):
            kinds.setdefault(fn, set()).add(inst.split()[-1] == "nt")
    assert len(kinds) == 3 and all(k == {True, False} for k in kinds.values()), kinds
