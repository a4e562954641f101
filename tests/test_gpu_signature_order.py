"""GPU parity of signatures read back from runs with seed groups: more words per
node than one pass through LDS takes, node counts around a block, both storage
orders, host and device destinations, one graph and a batch."""
import numpy as np
import pytest

import oracle
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp
from hipmem import DeviceArray

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 256, 257, 700])
@pytest.mark.parametrize("s,groups,order", [(64, 2, 0), (130, 3, 1), (700, 2, 1), (1100, 5, 0), (1100, 40, 1)])
@pytest.mark.parametrize("keep_order", [False, True])
def test_regrouped_signatures(n, s, groups, order, keep_order):
    rng = np.random.default_rng(n + s)
    src, dst = (rng.integers(0, n, 4 * n).astype(np.int32) for _ in range(2))
    seeds = rng.integers(0, n, s).astype(np.int32)
    print("signatures", n, s, groups, order, keep_order, flush=True)
    want = [oracle.propagate(n, src, dst, seeds[i:i + 512], False, final_sig=True)["final_sig"] for i in range(0, s, 512)]
    want = np.concatenate(want, axis=1)
    G = pp.pp_csr_build(n, src, dst, keep_order=keep_order)
    r = pp.pp_seeds_init(G, seeds, opts=pp.options(seed_groups=groups, seed_order=order))
    pp.pp_propagate_until_converged(r)
    host = pp.pp_get_signatures(r)
    assert np.array_equal(host[:, :want.shape[1]], want) and not host[:, want.shape[1]:].any()
    dev = DeviceArray(dtype=np.uint64, count=n * r.words)
    pp.pp_get_signatures(r, out=dev)
    assert np.array_equal(dev.to_host().reshape(host.shape), host)


def test_regrouped_signatures_of_a_batch():
    graphs = [gen.rmat(7, 6, 1), gen.path_graph(301), gen.grid_graph(11, 13)]
    seeds = [gen.sample_seeds(g.n, 100, 20 + i) for i, g in enumerate(graphs)]
    n, src, dst, offs, sd = gen.union_of(graphs, seeds)
    G = pp.pp_csr_build(n, src, dst, node_offsets=offs)
    r = pp.pp_seeds_init(G, sd, s=100, opts=pp.options(seed_groups=3, seed_order=1))
    pp.pp_propagate_until_converged(r)
    sig = pp.pp_get_signatures(r)
    for g, s, a, b in zip(graphs, seeds, offs, offs[1:]):
        want = oracle.propagate(g.n, g.src, g.dst, s, g.undirected, final_sig=True)["final_sig"]
        assert np.array_equal(sig[a:b], want)
