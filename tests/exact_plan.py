"""The exact interpolation's choice of form (csrc/exact_plan.h), compiled for
the host: what a call of these sizes takes in a workspace of these bytes."""
from __future__ import annotations

import ctypes
import functools
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1501_02565_amd", "csrc")
FIELDS = ("rounds", "big_groups", "pool_cap", "scratch_words", "cu", "ctl", "pend0", "pend1", "wide", "big",
          "bcount", "offset", "scratch", "meta", "order", "pool")
WRAP = """
#include "exact_plan.h"
extern "C" void plan(int H, int W, int N, int K, size_t begin, size_t used, size_t tail, long long* o) {
    const epic::ExactPlan p = epic::exact_plan(H, W, N, K, begin, used, tail);
    const long long v[] = {p.rounds, p.big_groups, (long long)p.pool_cap, (long long)p.scratch_words,
                           (long long)p.cu, (long long)p.ctl, (long long)p.pend[0], (long long)p.pend[1],
                           (long long)p.wide, (long long)p.big, (long long)p.bcount, (long long)p.offset,
                           (long long)p.scratch, (long long)p.meta, (long long)p.order, (long long)p.pool};
    for (unsigned i = 0; i < sizeof(v) / sizeof(v[0]); ++i) o[i] = v[i];
}
"""


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(WRAP)
        subprocess.check_call(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-fPIC", "-shared", "-I", CSRC,
                               "-o", so, src])
        lib = ctypes.CDLL(so)
    lib.plan.argtypes = [ctypes.c_int] * 4 + [ctypes.c_size_t] * 3 + [ctypes.POINTER(ctypes.c_longlong)]
    return lib


def plan_at(H, W, N, K, begin, used, tail):
    out = (ctypes.c_longlong * len(FIELDS))()
    _lib().plan(H, W, N, K, begin, used, tail, out)
    return dict(zip(FIELDS, out))


def up(v):
    return -(-v // 256) * 256


def lists_bytes(H, W, N, K):
    """What the call keeps at the workspace's end."""
    return up(8 * K * H * W) + up(N) + up(4 * H * W) + 2 * up(4 * N * K) + 2 * up(16 << 10) + 256


def plan(ws, H, W, N, K):
    """The plan of a call in a context of ws bytes."""
    import paper_1501_02565_amd as epic
    # a 1 x 1 workspace is the fixed head, five tile arrays and a pair: 1024
    # hash slots of 28 bytes and eleven small arrays
    fixed = epic.workspace_bytes(1, 1, 1, 1) - 5 * 256 - 1024 * 28 - 11 * 256
    assert fixed % 256 == 0
    tail = (ws - (lists_bytes(H, W, N, K) - 256)) // 256 * 256
    return plan_at(H, W, N, K, fixed, epic.workspace_bytes(H, W, N, K), tail)
