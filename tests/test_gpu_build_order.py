"""The storage order found on the device against the host's searches, array for
array: several searches in one graph (components with hubs of their own, nodes
that only a later root reaches, hubs that block a search), ties in degree, and
graphs whose searches are too deep for the device's passes."""
import numpy as np
import pytest

from hipmem import DeviceArray
from paper_2301_06499_amd import inputs as gen
from paper_2301_06499_amd import pp

pytestmark = pytest.mark.gpu


def hub_chain(hubs, leaves, tail, rng):
    """Hubs with `leaves` predecessors each, joined through ordinary nodes, every
    hub with a directed tail of `tail` nodes behind it, and stray nodes."""
    src, dst, n = [], [], 0
    for h in range(hubs):
        hub = n
        n += 1 + leaves + tail
        src += range(hub + 1, hub + 1 + leaves)
        dst += [hub] * leaves
        chain = [hub] + list(range(hub + 1 + leaves, hub + 1 + leaves + tail))
        src += chain[:-1]
        dst += chain[1:]
        if h:
            src += [hub + 1, chain[-1]]
            dst += [hub - 1, max(0, hub - 7)]
    n += 5
    extra = rng.integers(0, n, (2, n // 2))
    return n, np.array(src + extra[0].tolist(), np.int32), np.array(dst + extra[1].tolist(), np.int32)


def rmat(scale, ef, seed, extra=0):
    g = gen.rmat(scale, ef, seed)
    return g.n + extra, g.src, g.dst


def blocks(k, rng):
    parts = [rmat(8, 12, 30 + i) for i in range(k)]
    off = np.cumsum([0] + [p[0] for p in parts])
    src = np.concatenate([p[1] + o for p, o in zip(parts, off)])
    dst = np.concatenate([p[2] + o for p, o in zip(parts, off)])
    mix = rng.permutation(off[-1])
    return int(off[-1]), mix[src].astype(np.int32), mix[dst].astype(np.int32)


RNG = np.random.default_rng(7)
CASES = {
    "rmat": rmat(13, 16, 3, 77), "rmat sparse": rmat(14, 3, 4), "rmat dense": rmat(9, 60, 5),
    "blocks": blocks(9, RNG), "chain": hub_chain(12, 40, 3, RNG), "chain, long tails": hub_chain(3, 60, 300, RNG),
    "chain, deep": hub_chain(2, 30, 3000, RNG), "random": (4001,) + tuple(RNG.integers(0, 4001, (2, 30000)).astype(np.int32)),
    "two nodes": (2, np.array([0, 1], np.int32), np.array([1, 0], np.int32)),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("kw", [{}, {"undirected": True}, {"transpose": True}])
def test_device_order_equals_host_order(name, kw):
    n, src, dst = CASES[name]
    print("order", name, kw, "n", n, "pairs", len(src), flush=True)
    want = pp.pp_graph_get_csr(pp.pp_csr_build(n, src, dst, build="host", **kw))
    for s, d, build in ((src, dst, "device"), (DeviceArray(src), DeviceArray(dst), "auto")):
        got = pp.pp_graph_get_csr(pp.pp_csr_build(n, s, d, build=build, **kw))
        for field, x, y in zip(("rp", "col", "trp", "tcol", "perm"), want, got):
            assert np.array_equal(x, y), field
