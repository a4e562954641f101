"""GPU parity of rounds whose closing launch has one block or two:
lists of just under, exactly and just over one block's 256 words."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


def layers(width):
    """A node, three layers of width nodes (each node to its own and the next one's successor), a node."""
    a = np.arange(width, dtype=np.int32)
    src = [np.zeros(width, np.int32)]
    dst = [1 + a]
    for k in range(2):
        for shift in (0, 1):
            src.append(1 + k * width + a)
            dst.append(1 + (k + 1) * width + (a + shift) % width)
    src.append(1 + 2 * width + a)
    dst.append(np.full(width, 1 + 3 * width, np.int32))
    return 2 + 3 * width, np.concatenate(src), np.concatenate(dst)


@pytest.mark.parametrize("sched", [pp.PP_SCHED_PUSH, pp.PP_SCHED_PULL, pp.PP_SCHED_FUZZ])
@pytest.mark.parametrize("s,width", [(64, 255), (64, 256), (64, 257), (500, 31), (500, 32), (500, 33)])
def test_closing_blocks(s, width, sched):
    n, src, dst = layers(width)
    seeds = gen.sample_seeds(n, s, 3) if s <= n else np.arange(s, dtype=np.int32) % n
    seeds[0] = n - 1
    want = oracle.propagate(n, src, dst, seeds, False, seed_counts=True, final_sig=True)
    G = pp.pp_csr_build(n, src, dst)
    for sparse in (0, 1):
        r = pp.pp_seeds_init(G, seeds, opts=pp.options(scheduler=sched, seed_counts=True, node_stats=True,
                                                       fuzz_seed=5, sparse_pull=sparse))
        for again in range(2):
            counts, D = pp.pp_propagate_until_converged(r)
            assert int(D[0]) == want["D"] and list(counts[0]) == list(want["counts"])
            assert np.array_equal(pp.pp_get_seed_counts(r, want["D"] + 1)[0], want["seed_counts"])
            sig = pp.pp_get_signatures(r)
            assert np.array_equal(sig[:, :want["final_sig"].shape[1]], want["final_sig"])
            pp.pp_seeds_reset(r, seeds)
