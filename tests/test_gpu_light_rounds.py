"""GPU parity of the light rounds (small pushes one after the other in one
block) at the edges of their LDS capacities: a broom -- a path, a hub with K
leaves, a node behind each leaf -- whose hub pushes K + 1 arcs, whose leaves
make a frontier of K entries, and whose second ring pushes through K short
lists; K around H and LC = H / 2 of both block sizes (H = 4096 / W and
2048 / W)."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


def broom(K):
    path = np.arange(5, dtype=np.int32)
    leaves = np.arange(K, dtype=np.int32) + 6
    src = np.concatenate([path, np.full(K, 5, np.int32), leaves])
    dst = np.concatenate([path + 1, leaves, leaves + K])
    return 6 + 2 * K, src.astype(np.int32), dst.astype(np.int32)


def check(run, want):
    counts, D = pp.pp_propagate_until_converged(run)
    assert int(D[0]) == want["D"] and list(counts[0]) == list(want["counts"])
    sig = pp.pp_get_signatures(run)
    assert np.array_equal(sig[:, :want["final_sig"].shape[1]], want["final_sig"])
    assert np.array_equal(pp.pp_get_seed_counts(run, want["D"] + 1)[0], want["seed_counts"])


@pytest.mark.parametrize("s,W", [(3, 1), (100, 2), (250, 4), (500, 8)])
@pytest.mark.parametrize("edge", [1024, 2048, 4096])
@pytest.mark.parametrize("persistent", [False, True])
def test_light_capacities(s, W, edge, persistent):
    for K in (edge // W - 2, edge // W - 1, edge // W, edge // W + 1):
        n, src, dst = broom(K)
        seeds = np.concatenate([np.zeros(s // 2, np.int32), gen.sample_seeds(n, s - s // 2, K, distinct=False)])
        print("light", s, W, "K", K, "persistent", persistent, flush=True)
        want = oracle.propagate(n, src, dst, seeds, True, seed_counts=True, final_sig=True)
        G = pp.pp_csr_build(n, src, dst, undirected=True)
        for sched, plan in ((pp.PP_SCHED_PUSH, None), (pp.PP_SCHED_HEURISTIC, None),
                            (pp.PP_SCHED_PLAN, [1, 1, 1, 0, 1, 2, 1, 1, 0, 1, 1, 1])):
            r = pp.pp_seeds_init(G, seeds, opts=pp.options(scheduler=sched, seed_counts=True, persistent=persistent,
                                                           max_rounds=want["D"] + 4))
            if plan is not None:
                pp.pp_run_set_plan(r, plan)
                pp.pp_seeds_reset(r, seeds)
            check(r, want)
            modes, arcs = pp.pp_get_round_log(r, want["D"] + 2)
            assert modes[want["D"] + 1] >= 0 and modes[0] == pp.MODE_INIT
            pp.pp_seeds_reset(r, seeds)
            check(r, want)
