"""GPU parity of PROPAGATE-S at every row width and its edges: counts, D and
the arcs examined against the literal oracle."""
import functools

import numpy as np
import pytest

import oracle.propagate_s as ops
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu

# lists far longer than a wave's step, and one that a whole block walks; long
# passes; no arcs at all.  Node counts
# that are no multiple of 4 or 64, and seeds at 12 nodes only: the oracle runs
# once per node, and its figures add up over the seeds.
GRAPHS = {"rmat": (gen.rmat(9, 90, 3), 3), "path": (gen.path_graph(131), 0), "star": (gen.star_graph(9003), 2),
          "empty": (gen.Graph(5, np.zeros(0, np.int32), np.zeros(0, np.int32), False), 0)}


@functools.lru_cache(None)
def per_node(name):
    g, extra = GRAPHS[name]
    nodes = gen.sample_seeds(g.n + extra, 12, 5, distinct=False)
    return nodes, [ops.propagate_s(g.n + extra, g.src, g.dst, [x], g.undirected, stored=True) for x in nodes.tolist()]


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("s,concurrent", [(1, 0), (7, 0), (8, 0), (9, 0), (31, 0), (33, 17), (64, 0), (65, 64),
                                          (128, 0), (200, 0), (300, 300), (513, 513)])
def test_seq_rows(name, s, concurrent):
    g, extra = GRAPHS[name]
    nodes, alone = per_node(name)
    pick = np.random.default_rng(s).integers(0, len(nodes), s)
    print("seq rows", name, s, concurrent, flush=True)
    D = max(alone[i][1] for i in pick)
    want = np.zeros(D + 1, np.int64)
    for i in pick:
        want[:alone[i][1] + 1] += np.asarray(alone[i][0])[:alone[i][1] + 1]
    examined = sum(int(alone[i][2]) for i in pick)
    G = pp.pp_csr_build(g.n + extra, g.src, g.dst, undirected=g.undirected, keep_order=True)
    for call in (pp.pp_propagate_s, pp.pp_propagate_s_noalloc):
        counts, Dg, ex = call(G, nodes[pick], concurrent=concurrent)
        assert Dg == D and list(counts) == list(want) and ex == examined, call.__name__


def test_seq_rows_pass_limit():
    g = gen.path_graph(40)
    seeds = np.arange(16, dtype=np.int32)
    G = pp.pp_csr_build(g.n, g.src, g.dst, undirected=True)
    for cap in (1, 2, 9, 10):
        if cap == 1:
            counts, D, _ = pp.pp_propagate_s(G, seeds, cap_rounds=cap)
            assert list(counts) == [16] and D == 0
            continue
        with pytest.raises(pp.PPError) as e:
            pp.pp_propagate_s(G, seeds, cap_rounds=cap)
        assert e.value.code == pp.PP_ENOTCONV
