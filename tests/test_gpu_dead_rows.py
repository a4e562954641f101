"""Small graphs among many nodes without successors, rows beyond the caches: rounds
by the pull that leaves those rows alone, against the oracle on the graph's own
nodes."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,n", [(512, (1 << 21) + 5), (64, (1 << 24) + (1 << 18))])
@pytest.mark.parametrize("sched", [pp.PP_SCHED_HEURISTIC, pp.PP_SCHED_PULL, pp.PP_SCHED_FUZZ])
def test_small_graph_among_many_nodes(s, n, sched):
    g = gen.rmat(12, 8, 5)
    step = (n - 1) // (g.n - 1)   # the graph's nodes spread over all ids
    seeds = gen.sample_seeds(g.n, s, 4)
    print("dead rows", n, s, "sched", sched, flush=True)
    want = oracle.propagate(g.n, g.src, g.dst, seeds, False, final_sig=True)
    G = pp.pp_csr_build(n, g.src * step, g.dst * step)
    r = pp.pp_seeds_init(G, seeds * step, opts=pp.options(scheduler=sched, fuzz_seed=2, max_rounds=64))
    for _ in range(2):
        counts, D = pp.pp_propagate_until_converged(r)
        assert int(D[0]) == want["D"] and list(counts[0]) == list(want["counts"])
        sig = pp.pp_get_signatures(r)
        rows = sig[::step][:g.n]
        assert np.array_equal(rows[:, :want["final_sig"].shape[1]], want["final_sig"])
        assert np.count_nonzero(sig) == np.count_nonzero(rows)
        pp.pp_seeds_reset(r, seeds * step)
