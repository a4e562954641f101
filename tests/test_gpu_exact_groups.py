"""GPU parity of the exact neighbourhood function with its groups side by side:
ragged last groups, more groups than one run takes, and a run that the
allocator refuses, which falls back to one group at a time."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp
from hipmem import hip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def case():
    g = gen.rmat(12, 4, 9)
    n = g.n + 905
    total = np.zeros(64, np.int64)
    for first in range(0, n, 512):
        w = oracle.propagate(n, g.src, g.dst, np.arange(first, min(n, first + 512), dtype=np.int32), True)
        total[:w["D"] + 1] += np.asarray(w["counts"])
    return n, g, np.trim_zeros(total, "b")


@pytest.mark.parametrize("group", [1, 63, 64, 65, 500, 512])
@pytest.mark.parametrize("sched", [pp.PP_SCHED_HEURISTIC, pp.PP_SCHED_FUZZ])
def test_exact_groups(case, group, sched):
    n, g, want = case
    G = pp.pp_csr_build(n, g.src, g.dst, undirected=True)
    print("exact groups", group, sched, flush=True)
    counts, D = pp.pp_exact_counts(G, group=group, opts=pp.options(scheduler=sched, fuzz_seed=2), cap_rounds=64)
    assert list(counts) == list(want) and D == len(want) - 1


def test_exact_groups_without_memory(case):
    n, g, want = case
    G = pp.pp_csr_build(n, g.src, g.dst, undirected=True)
    refused = []

    def alloc(nbytes, stream):
        if nbytes > 2 << 20:
            refused.append(nbytes)
            return 0
        p = ctypes.c_void_p()
        return p.value if hip().hipMalloc(ctypes.byref(p), nbytes) == 0 else 0

    pp.pp_set_allocator(alloc, lambda p, st: hip().hipFree(ctypes.c_void_p(p)))
    try:
        counts, D = pp.pp_exact_counts(G, group=512, cap_rounds=64)
    finally:
        pp.pp_set_allocator(None, None)
    assert refused and list(counts) == list(want) and D == len(want) - 1
