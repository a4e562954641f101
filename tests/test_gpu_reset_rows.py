"""GPU parity after resets to other seeds: the old seeds' rows are cleared by the
blocks behind the reset's fills, for few and many groups (one fill launch holds
32 segments) and lists of just under and over one block's 256 seeds."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,groups", [(255, 0), (256, 0), (257, 0), (130, 2), (700, 2), (300, 9), (300, 10), (300, 24)])
def test_reset_to_other_seeds(s, groups):
    g = gen.rmat(10, 6, 4)
    G = pp.pp_csr_build(g.n, g.src, g.dst)
    r = None
    for k in range(4):
        seeds = gen.sample_seeds(g.n, s, 20 + k)
        want = oracle.propagate(g.n, g.src, g.dst, seeds, False, seed_counts=True, final_sig=True)
        if r is None:
            r = pp.pp_seeds_init(G, seeds, opts=pp.options(seed_counts=True, seed_groups=groups, max_rounds=64))
        else:
            pp.pp_seeds_reset(r, seeds)
        counts, D = pp.pp_propagate_until_converged(r)
        assert int(D[0]) == want["D"] and list(counts[0]) == list(want["counts"])
        assert np.array_equal(pp.pp_get_seed_counts(r, want["D"] + 1)[0], want["seed_counts"])
        sig = pp.pp_get_signatures(r)
        assert np.array_equal(sig[:, :want["final_sig"].shape[1]], want["final_sig"])
