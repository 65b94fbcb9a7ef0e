"""Inline assembly that writes M0 says so: the compiler keeps its own values there
(indexed register moves, LDS loads of its own), and would use a stale one after an
undeclared write."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_writes_of_m0_are_declared():
    found = 0
    for path in glob.glob(os.path.join(ROOT, "paper_2605_27255_amd", "csrc", "*.h*")):
        for stmt in re.findall(r"asm\s+volatile\s*\((.*?)\);", open(path).read(), re.S):
            if re.search(r"\bs_\w+\s+m0\b", stmt):
                found += 1
                assert '"m0"' in stmt.rsplit(":", 1)[1], (path, stmt)
    assert found
