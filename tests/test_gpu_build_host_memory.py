"""A device build whose host part finds no memory (the offsets for the host's
searches, or the numbering that the device found) reports PP_ENOMEM; no exception
crosses the C interface, and the library goes on.  In a child process, whose
address space is limited for the call; device memory comes from a block taken
before."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.gpu

CHILD = r"""
import ctypes, resource, sys
import numpy as np
sys.path[:0] = [%(root)r, %(root)r + "/tests"]
from hipmem import hip
from paper_2301_06499_amd import pp
n, hot = 1 << 26, %(hot)d
POOL = 8 << 30
base, used = ctypes.c_void_p(), 0
assert hip().hipMalloc(ctypes.byref(base), POOL) == 0
def alloc(size, stream):
    global used
    at = used
    used += (size + 255) & ~255
    return base.value + at if used <= POOL else 0
pp.pp_set_allocator(alloc, lambda p, st: None)
src = np.arange(64, dtype=np.int32) + 1
dst = np.zeros(64, np.int32) if hot else src * 1000
def build(nodes):
    global used
    used = 0
    pp.pp_csr_build(nodes, src, dst, build="device").free()
build(1 << 17)   # kernels loaded, streams and staging made
size = next(int(l.split()[1]) << 10 for l in open("/proc/self/status") if l.startswith("VmSize"))
soft, hard = resource.getrlimit(resource.RLIMIT_AS)
resource.setrlimit(resource.RLIMIT_AS, (size + (160 << 20), hard))
try:
    build(n)
    code = 0
except pp.PPError as e:
    code = e.code if "host memory for the storage order" in str(e) else -99
resource.setrlimit(resource.RLIMIT_AS, (soft, hard))
print("limited build:", code, flush=True)
assert code == pp.PP_ENOMEM
build(n)
print("done", flush=True)
"""


@pytest.mark.parametrize("hot", [0, 1])
def test_no_host_memory_is_reported(hot):
    out = subprocess.run([sys.executable, "-u", "-c", CHILD % {"root": ROOT, "hot": hot}], capture_output=True, text=True,
                         timeout=100)
    print(out.stdout, out.stderr[-2000:], flush=True)
    assert out.returncode == 0 and "done" in out.stdout
