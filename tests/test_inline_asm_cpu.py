"""Inline assembly of the kernels: a statement that writes m0 says so, so that
the compiler moves no use of its own across it."""
import glob
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1602_05901_amd", "csrc")


def statements(text):
    for m in re.finditer(r"\basm\s+volatile\s*\(", text):
        depth, at = 1, m.end()
        while depth:
            depth += {"(": 1, ")": -1}.get(text[at], 0)
            at += 1
        yield text[m.start():at]


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.h*"))), ids=os.path.basename)
def test_m0_is_named(path):
    with open(path) as f:
        for s in statements(f.read()):
            if re.search(r"\bs_\w+\s+m0\b", s):
                assert re.search(r'"m0"\s*\)$', s), s
