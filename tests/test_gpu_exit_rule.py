"""Early-exit pulls are given up where they gather most arcs all the same -- a ring
whose neighbours lack the same bits -- and not where they pay; outputs against the
oracle either way."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


def ring(n, k):
    i = np.arange(n, dtype=np.int64)
    src = np.concatenate([i] * k)
    dst = np.concatenate([(i + j) % n for j in range(1, k + 1)])
    return n, src.astype(np.int32), dst.astype(np.int32)


@pytest.mark.parametrize("s,sched", [(30, pp.PP_SCHED_PULL), (250, pp.PP_SCHED_PULL), (250, pp.PP_SCHED_HEURISTIC)])
def test_ring(s, sched):
    n, src, dst = ring(70_001, 8)
    seeds = gen.sample_seeds(n, s, 3)
    print("exit rule ring", s, sched, flush=True)
    want = oracle.propagate(n, src, dst, seeds, True, final_sig=True)
    G = pp.pp_csr_build(n, src, dst, undirected=True)
    assert G.arcs >= 1 << 20
    r = pp.pp_seeds_init(G, seeds, opts=pp.options(scheduler=sched))
    counts, D = pp.pp_propagate_until_converged(r)
    assert int(D[0]) == want["D"] and list(counts[0]) == list(want["counts"])
    assert np.array_equal(pp.pp_get_signatures(r)[:, :want["final_sig"].shape[1]], want["final_sig"])
    modes, _ = pp.pp_get_round_log(r, want["D"] + 2)
    pulls, exits = int((modes == pp.MODE_PULL).sum()), pp.pp_get_path_counts(r)[0]
    print("pulls", pulls, "early exits", exits, flush=True)
    assert exits <= pulls // 4
    assert sched == pp.PP_SCHED_HEURISTIC or (pulls >= 40 and exits >= 1)


def test_random_graph():
    g = gen.erdos_renyi_gnm(1 << 18, 1 << 20, 3)
    seeds = gen.sample_seeds(g.n, 256, 3)
    G = pp.pp_csr_build(g.n, g.src, g.dst, undirected=True)
    r = pp.pp_seeds_init(G, seeds, opts=pp.options())
    _, D = pp.pp_propagate_until_converged(r)
    modes, _ = pp.pp_get_round_log(r, int(D[0]) + 2)
    print("pulls", int((modes == pp.MODE_PULL).sum()), pp.pp_get_path_counts(r), flush=True)
    assert pp.pp_get_path_counts(r)[0] >= 2
