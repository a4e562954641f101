"""The rounds take the paths they are meant to: early-exit pulls and what they
leave to chunks, light rounds up to their capacity and not past it, and steps
that only list a frontier -- on the graphs whose outputs the tests of those paths
compare."""
import numpy as np
import pytest

from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp
from test_gpu_early_exit import graph as exit_graph
from test_gpu_light_rounds import broom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,groups,sparse", [(64, 0, 0), (200, 0, 0), (256, 0, 1), (512, 3, 0)])
def test_early_exit_pulls_run(s, groups, sparse):
    n, src, dst = exit_graph(37)
    seeds = gen.sample_seeds(1 << 16, s, 5)
    seeds[s // 2:s // 2 + 3] = [n - 1, n - 20, n - 1][:len(seeds[s // 2:s // 2 + 3])]   # on the path
    G = pp.pp_csr_build(n, src, dst)
    r = pp.pp_seeds_init(G, seeds, opts=pp.options(scheduler=pp.PP_SCHED_PULL, max_rounds=64, sparse_pull=sparse,
                                                   seed_groups=groups))
    pp.pp_propagate_until_converged(r)
    counts = [pp.pp_get_path_counts(r, j) for j in range(r.groups)]
    assert all(c[0] >= 2 for c in counts), counts
    assert any(c[1] >= 100 for c in counts), counts   # nodes that walked past EXIT_LIMIT arcs
    assert all(c[2:] == (0, 0) for c in counts), counts
    pp.pp_seeds_reset(r, seeds)
    assert pp.pp_get_path_counts(r) == (0, 0, 0, 0)


@pytest.mark.parametrize("s,W", [(3, 1), (100, 2), (250, 4), (500, 8)])
@pytest.mark.parametrize("persistent,H", [(False, 4096), (True, 2048)])
def test_light_rounds_run_up_to_their_capacity(s, W, persistent, H):
    """All seeds at the path's end: the hub's round pushes K + 1 arcs of one node,
    the next one K nodes' lists."""
    got = {}
    for K in (H // (2 * W) - 8, 2 * H // W):
        n, src, dst = broom(K)
        seeds = np.zeros(s, np.int32)
        G = pp.pp_csr_build(n, src, dst, undirected=True)
        r = pp.pp_seeds_init(G, seeds, opts=pp.options(scheduler=pp.PP_SCHED_PUSH, persistent=persistent, max_rounds=64))
        _, D = pp.pp_propagate_until_converged(r)
        got[K] = int(D[0]) + 1 - pp.pp_get_path_counts(r)[2]
    print("rounds that were not light", s, persistent, got, flush=True)
    assert got[H // (2 * W) - 8] <= 2   # the leaves' lists hold twice as many arcs
    assert got[2 * H // W] >= 2         # the hub's round, and the leaves'


def test_listing_steps_run():
    g = gen.grid_graph(37, 41)
    seeds = gen.sample_seeds(g.n, 20, 5)
    G = pp.pp_csr_build(g.n, g.src, g.dst, undirected=True)
    opts = pp.options(scheduler=pp.PP_SCHED_FUZZ, fuzz_seed=5)
    r = pp.pp_seeds_init(G, seeds, opts=opts)
    _, D = pp.pp_propagate_until_converged(r)
    modes, _ = pp.pp_get_round_log(r, int(D[0]) + 2)
    after_pull = sum(modes[q] != pp.MODE_PULL and modes[q - 1] == pp.MODE_PULL for q in range(2, len(modes)))
    assert pp.pp_get_path_counts(r)[3] == after_pull > 0
    single = pp.pp_seeds_init(G, seeds, opts=opts)
    while not pp.pp_propagate_round(single)[1]:
        pass
    assert pp.pp_get_path_counts(single) == (0, 0, 0, 0)   # rounds of three launches


def test_which_is_checked():
    g = gen.path_graph(10)
    G = pp.pp_csr_build(g.n, g.src, g.dst, undirected=True)
    r = pp.pp_seeds_init(G, np.array([0], np.int32))
    for which in (-1, 1):
        with pytest.raises(pp.PPError) as e:
            pp.pp_get_path_counts(r, which)
        assert e.value.code == pp.PP_EINVAL
