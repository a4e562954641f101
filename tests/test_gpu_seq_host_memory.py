"""PROPAGATE-S with a long table of counts: the call's own host memory follows the
passes it runs, not the table's length."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.gpu

CHILD = r"""
import ctypes, resource, sys
import numpy as np
sys.path[:0] = [%r]
from paper_2301_06499_amd import inputs as gen, pp
g = gen.path_graph(40)
G = pp.pp_csr_build(g.n, g.src, g.dst, undirected=True)
seeds = np.arange(16, dtype=np.int32)
counts = np.full(1 << 27, 7, np.int64)   # 1 GiB, resident
ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
D, examined = ctypes.c_int32(), ctypes.c_int64()
def call(cap):
    assert pp.lib().pp_propagate_s(G.handle, ptr(seeds), 16, 0, None, ptr(counts), cap, ctypes.byref(D), ctypes.byref(examined)) == 0
    assert D.value == 39 and counts[0] == 16 and counts[1] == 31 and not counts[40:cap].any()
call(64)
before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
call(1 << 27)
grown = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before
print("grown by", grown, "KiB", flush=True)
assert grown < 256 << 10
"""


def test_host_memory_follows_the_passes():
    out = subprocess.run([sys.executable, "-u", "-c", CHILD % ROOT], capture_output=True, text=True, timeout=100)
    print(out.stdout, out.stderr[-2000:], flush=True)
    assert out.returncode == 0
