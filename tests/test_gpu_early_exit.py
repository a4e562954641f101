"""GPU parity of the pulls that stop each list early, at sizes where they run
(2^20 stored arcs and up), against the CPU oracle, bit for bit.

The graph is an R-MAT with long lists beside a path that no R-MAT node
reaches: while the path's seeds still spread, their bits are live, so every
R-MAT node lacks a live bit and walks its whole list -- through the chunks
that a node leaves after EXIT_LIMIT arcs -- and the node count is no multiple
of a wave's 64 nodes.
"""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


def graph(path_nodes):
    g = gen.rmat(16, 26, 7)
    i = np.arange(path_nodes - 1, dtype=np.int32) + g.n
    return g.n + path_nodes, np.concatenate([g.src, i]), np.concatenate([g.dst, i + 1])


@pytest.mark.parametrize("s,groups,sched,sparse,pull_k", [
    (1, 0, pp.PP_SCHED_PULL, 0, 4), (64, 0, pp.PP_SCHED_PULL, 0, 4), (65, 0, pp.PP_SCHED_PULL, 0, 2),
    (200, 0, pp.PP_SCHED_PULL, 0, 4), (300, 0, pp.PP_SCHED_PULL, 0, 4), (512, 3, pp.PP_SCHED_PULL, 0, 4),
    (100, 0, pp.PP_SCHED_FUZZ, 0, 4), (256, 0, pp.PP_SCHED_FUZZ, 1, 4), (256, 0, pp.PP_SCHED_FUZZ, 2, 4),
    (512, pp.PP_GROUPS_BY_REACH, pp.PP_SCHED_HEURISTIC, 0, 4)])
def test_early_exit_pulls(s, groups, sched, sparse, pull_k):
    n, src, dst = graph(37)
    seeds = gen.sample_seeds(1 << 16, s, 5)
    seeds[s // 2:s // 2 + 3] = [n - 1, n - 20, n - 1][:len(seeds[s // 2:s // 2 + 3])]   # on the path
    print("early exit s", s, "groups", groups, "sched", sched, "sparse_pull", sparse, "pull_k", pull_k, flush=True)
    want = oracle.propagate(n, src, dst, seeds, False, seed_counts=True, final_sig=True)
    G = pp.pp_csr_build(n, src, dst)
    assert G.arcs >= 1 << 20
    r = pp.pp_seeds_init(G, seeds, opts=pp.options(scheduler=sched, seed_counts=True, max_rounds=64, fuzz_seed=3,
                                                   sparse_pull=sparse, pull_k=pull_k, seed_groups=groups))
    for again in range(2):   # a reset clears what the early-exit rounds left
        counts, D = pp.pp_propagate_until_converged(r)
        assert int(D[0]) == want["D"] and list(counts[0]) == list(want["counts"])
        assert np.array_equal(pp.pp_get_seed_counts(r, want["D"] + 1)[0], want["seed_counts"])
        sig = pp.pp_get_signatures(r)
        assert np.array_equal(sig[:, :want["final_sig"].shape[1]], want["final_sig"])
        assert not sig[:, want["final_sig"].shape[1]:].any()
        modes, arcs = pp.pp_get_round_log(r, want["D"] + 2)
        pulls = [q for q in range(1, want["D"] + 2) if modes[q] == pp.MODE_PULL]
        assert pulls and (groups or all(arcs[q] == G.arcs for q in pulls))
        pp.pp_seeds_reset(r, seeds)
