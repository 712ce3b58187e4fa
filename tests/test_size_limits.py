"""The largest number of matches: the edge hash has 16 slots a match, whose
power of two must fit an int.  Above 2^26 the sizing never returned."""
from __future__ import annotations

import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
import paper_1501_02565_amd._lib as l
L = l.load()
P = 0x1000
def both(n):
    return L.epic_workspace_bytes(16, 16, n, 4, 1, 0), L.epic_validate(P, 16, 16, P, n, 4, 1.0, 1, P)
b, v = both(1 << 26)
assert v == l.OK and 28 << 30 <= b < 64 << 30, (b, v)
for n in ((1 << 26) + 1, 1 << 27, (1 << 30) - 1, (1 << 31) - 1):
    assert both(n) == (0, l.ERR_ARG), n
print("ok")
"""


def test_matches_above_2_26_are_refused():
    # in a process of its own, so that a call that does not return ends
    out = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=60, cwd=ROOT)
    assert out.returncode == 0 and out.stdout.strip().endswith("ok"), out.stderr
