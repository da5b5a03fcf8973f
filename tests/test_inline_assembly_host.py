"""Inline assembly in the kernels names no scalar registers: the compiler keeps the distance that the hardware wants between a write of a
scalar register and a memory instruction that reads it, but it does not look at the operands of an asm statement."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_22036_amd", "csrc")
SOURCES = sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")))


def statements(path):
    text = re.sub(r"//[^\n]*", "", open(path).read())
    return re.findall(r"\basm\s*(?:volatile)?\s*\((.*?)\)\s*;", text, flags=re.S)


def test_statements_are_found():
    assert len([s for p in SOURCES for s in statements(p) if "global_store_dwordx4" in s]) >= 3


@pytest.mark.parametrize("path", SOURCES, ids=os.path.basename)
def test_no_scalar_operands(path):
    for s in statements(path):
        constraints = re.findall(r'"([^"]*)"\s*\(', s)
        assert all("s" not in c and "r" not in c for c in constraints), s
