"""GPU parity of propagations that stop at a round limit and go on from there."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


def check(run, want):
    counts, D = pp.pp_propagate_until_converged(run)
    assert int(D[0]) == want["D"] and list(counts[0]) == list(want["counts"])
    sig = pp.pp_get_signatures(run)
    assert np.array_equal(sig[:, :want["final_sig"].shape[1]], want["final_sig"])
    assert np.array_equal(pp.pp_get_seed_counts(run, want["D"] + 1)[0], want["seed_counts"])


@pytest.mark.parametrize("persistent", [False, True])
def test_round_limits_and_snapshots(persistent):
    """Rounds up to a limit, the rest after it; a full log; a snapshot taken between."""
    g = gen.path_graph(300)
    seeds = gen.sample_seeds(g.n, 20, 4)
    want = oracle.propagate(g.n, g.src, g.dst, seeds, True, seed_counts=True, final_sig=True)
    G = pp.pp_csr_build(g.n, g.src, g.dst, undirected=True)
    opts = pp.options(seed_counts=True, persistent=persistent)
    r = pp.pp_seeds_init(G, seeds, opts=opts)
    counts, D = pp.pp_propagate_until_converged(r, max_rounds=11, raise_on_cap=False)
    assert r.round == 12 and list(counts[0]) == list(want["counts"][:12])
    snap = pp.pp_run_snapshot(r)
    check(r, want)
    check(snap, want)
    short = pp.pp_seeds_init(G, seeds, opts=pp.options(persistent=persistent, max_rounds=17))
    with pytest.raises(pp.PPError) as e:
        pp.pp_propagate_until_converged(short)
    assert e.value.code == pp.PP_ENOTCONV
    counts, D = pp.pp_propagate_until_converged(short, raise_on_cap=False)
    assert list(counts[0]) == list(want["counts"][:18])
