"""Inline assembly of the kernels (host code, no GPU): only scalar, wait, barrier
and memory instructions.  The compiler does not look inside an assembly
string, so it inserts none of the wait states that a vector instruction needs
after the MFMA that produces its operand; vector arithmetic is left to
expressions and builtins."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_02043_amd", "csrc")
ALLOWED = {"s_nop", "s_waitcnt", "s_barrier", "s_getreg_b32", "global_load_lds_dwordx4"}


def mnemonics(text):
    """Mnemonics of every asm statement of a source text."""
    found = []
    for m in re.finditer(r"\basm\s*(?:volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", text.replace("\\\n", " ")):
        body = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
        found += [line.split()[0] for line in body.replace("\\t", " ").split("\\n") if line.split()]
    return found


def test_the_scan_sees_vector_arithmetic():
    assert mnemonics('asm("v_max3_f32 %0, %1" : "=v"(r));\nasm volatile("" : "+v"(t));') == ["v_max3_f32"]
    assert mnemonics('asm volatile(\n "s_nop 0\\n\\t"\n "v_add_f32 %0\\n" :::);') == ["s_nop", "v_add_f32"]


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.hip"))), ids=os.path.basename)
def test_no_vector_arithmetic_in_assembly(path):
    with open(path) as f:
        found = mnemonics(f.read())
    assert found, "no assembly found: the scan no longer reads this file"
    assert set(found) <= ALLOWED, sorted(set(found) - ALLOWED)
