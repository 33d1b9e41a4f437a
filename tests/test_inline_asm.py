"""Inline assembly of the kernels says what it writes: m0, which the compiler otherwise believes to hold what it set last."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_assembly_that_writes_m0_declares_it():
    found = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2602_03495_amd", "csrc", "*"))):
        for stmt in re.findall(r"\basm\b.*?;", open(path).read(), flags=re.S):
            if re.search(r"\bs_mov_b32 m0\b", stmt):
                found += 1
                assert '"m0"' in stmt.rsplit(":", 1)[1], (path, stmt)
    assert found > 0
