"""Resets of a snapshot: the copy has its own room for the stored ids of device
seeds, on both engines, and clears what its last seeds left."""
import numpy as np
import pytest

import oracle
from hipmem import DeviceArray
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


def check(run, g, seeds, offs, s):
    counts, D = pp.pp_propagate_until_converged(run)
    sig = pp.pp_get_signatures(run)
    for k in range(len(offs) - 1):
        lo, hi = offs[k], offs[k + 1]
        mine = (g.src >= lo) & (g.src < hi)
        want = oracle.propagate(hi - lo, g.src[mine] - lo, g.dst[mine] - lo, seeds[k * s:(k + 1) * s] - lo, False,
                                final_sig=True)
        assert int(D[k]) == want["D"] and list(counts[k][:want["D"] + 1]) == list(want["counts"][:want["D"] + 1])
        assert np.array_equal(sig[lo:hi, :want["final_sig"].shape[1]], want["final_sig"])


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("graphs", [1, 3])
@pytest.mark.parametrize("s", [5, 70])
def test_reset_of_a_copy(persistent, graphs, s):
    parts = [gen.rmat(9, 8, 40 + k) for k in range(graphs)]
    offs = np.cumsum([0] + [p.n for p in parts])
    g = gen.Graph(int(offs[-1]), np.concatenate([p.src + o for p, o in zip(parts, offs)]).astype(np.int32),
                  np.concatenate([p.dst + o for p, o in zip(parts, offs)]).astype(np.int32), False, "batch")
    sets = [np.concatenate([gen.sample_seeds(p.n, s, 7 * k + q) + o for q, (p, o) in enumerate(zip(parts, offs))])
            .astype(np.int32) for k in range(4)]
    G = pp.pp_csr_build(g.n, g.src, g.dst, node_offsets=offs if graphs > 1 else None)
    r = pp.pp_seeds_init(G, sets[0], s=s, opts=pp.options(persistent=persistent))
    copy = pp.pp_run_snapshot(r)
    print("snapshot reset", "persistent" if persistent else "rounds", graphs, s, flush=True)
    check(copy, g, sets[0], offs, s)
    for seeds in sets[1:]:   # device seeds, host seeds, device seeds
        placed = DeviceArray(seeds) if seeds is not sets[2] else seeds
        pp.pp_seeds_reset(copy, placed)
        check(copy, g, seeds, offs, s)
    check(r, g, sets[0], offs, s)
