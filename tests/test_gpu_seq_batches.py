"""PROPAGATE-S with rows for more seeds than are in flight: the same counts as
PROPAGATE-P, on every entry point, and in the promised memory where the larger
rows find none."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp
from test_gpu_allocator import CountingAllocator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [513, 4000])
@pytest.mark.parametrize("n", [300, 5000])
def test_more_seeds_than_a_row_holds(n, s):
    """A tiny graph takes them seed by seed in one batch, a larger one row by row."""
    g = gen.erdos_renyi_gnm(n, 3 * n, 4)
    seeds = np.resize(gen.sample_seeds(g.n, 64, 6), s)
    one = oracle.propagate(g.n, g.src, g.dst, seeds[:64], True, seed_counts=True)
    per = np.asarray(one["seed_counts"], np.int64)
    want = per.sum(1) * (s // 64) + per[:, :s % 64].sum(1)
    G = pp.pp_csr_build(g.n, g.src, g.dst, undirected=True)
    print("seq many", n, s, flush=True)
    ex = [pp.pp_propagate_s(G, seeds, concurrent=c, cap_rounds=64)[2] for c in (7, 100)]
    counts, D, examined = pp.pp_propagate_s(G, seeds, concurrent=s, cap_rounds=64)
    assert D == one["D"] and list(counts) == list(want) and [examined] * 2 == ex


@pytest.mark.parametrize("s", [8, 9, 15, 31, 130, 255, 257])
def test_partly_filled_rows(s):
    g = gen.rmat(11, 8, 9)
    seeds = gen.sample_seeds(g.n, s, s)
    print("seq batches", s, flush=True)
    want = oracle.propagate(g.n, g.src, g.dst, seeds, False)
    G = pp.pp_csr_build(g.n, g.src, g.dst)
    _, _, examined = pp.pp_propagate_s(G, seeds, concurrent=7)   # seed-major
    calls = [lambda c=c: pp.pp_propagate_s(G, seeds, concurrent=c, cap_rounds=64) for c in (0, s)]
    calls.append(lambda: pp.pp_propagate_s_noalloc(G, seeds, cap_rounds=64))
    for call in calls:
        counts, D, ex = call()
        assert D == want["D"] and list(counts) == list(want["counts"]) and ex == examined
    # no memory for the larger rows: the promised amount will do
    a = CountingAllocator()
    promised = 16 * min(s, 256) * ((g.n + 63) // 64) + 8 * 64 + 8 * 256 + 40 * 256
    pp.pp_set_allocator(lambda n, st: a.alloc(n, st) if n <= promised else 0, a.release)
    try:
        counts, D, ex = calls[0]()
    finally:
        pp.pp_set_allocator(None, None)
    assert D == want["D"] and list(counts) == list(want["counts"]) and ex == examined and a.live == {}
