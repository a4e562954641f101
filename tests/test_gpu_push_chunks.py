"""GPU parity of pushes around the number of chunks of long predecessor lists
from which the words are read before the atomics (16384 chunks)."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


# chunks hold 256 words: 512 predecessors are 16 chunks of eight words, 8 of four, 2 of one
@pytest.mark.parametrize("s,hubs", [(500, 1023), (500, 1024), (200, 2048), (64, 8191), (64, 8192)])
def test_push_chunks(s, hubs):
    """The last node's seeds reach every hub in round 1 and, by 512 predecessors each, every node in round 2."""
    a = np.repeat(np.arange(512, dtype=np.int32), hubs)
    b = np.tile(512 + np.arange(hubs, dtype=np.int32), 512)
    n = 512 + hubs + 1
    src = np.concatenate([a, 512 + np.arange(hubs, dtype=np.int32)])
    dst = np.concatenate([b, np.full(hubs, n - 1, np.int32)])
    seeds = np.full(s, n - 1, np.int32)
    seeds[::3] = gen.sample_seeds(n, s, 4)[::3]
    want = oracle.propagate(n, src, dst, seeds, False, seed_counts=True, final_sig=True)
    G = pp.pp_csr_build(n, src, dst)
    r = pp.pp_seeds_init(G, seeds, opts=pp.options(scheduler=pp.PP_SCHED_PUSH, seed_counts=True))
    for again in range(2):
        counts, D = pp.pp_propagate_until_converged(r)
        assert int(D[0]) == want["D"] and list(counts[0]) == list(want["counts"])
        assert np.array_equal(pp.pp_get_seed_counts(r, want["D"] + 1)[0], want["seed_counts"])
        sig = pp.pp_get_signatures(r)
        assert np.array_equal(sig[:, :want["final_sig"].shape[1]], want["final_sig"])
        pp.pp_seeds_reset(r, seeds)
