"""The work a user has this library do, as timed cases.

A program that measures graphs holds a graph (`pp_csr_build`) and a run
(`pp_seeds_init`), and then asks again and again: place a seed sample,
propagate it to convergence, read the counts (`sample` cases).  Beside that
it measures whole batches of graphs, the exact neighbourhood function, seeds
one at a time (PROPAGATE-S), a progressive sample, and a graph seen once
(`new_graph`: build, run, read).

The graphs are the families of this repository's own workloads: Erdos-Renyi
(10k nodes), R-MAT with edge factor 16 (directed, and undirected as a social
network is), square lattices with deleted edges and shortcuts (up to 4096 on a
side), and the uneven batch of R-MATs, lattices and paths.  R-MAT scale 24
stands for the graphs whose rows exceed the caches; scale 26, of the headline
benchmark, has the same kernels and bounds at four times the inputs.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2301_06499_amd import inputs, pp


def listed():
    return [
        # the smallest call: a 10k-node graph, one word of seeds; launches and waits
        _sample("er10k_s64", "er", n=10000, m=50000, undirected=True, s=64),
        # a social network (arcs both ways), a ragged seed count, and every
        # per-seed, per-node and signature output read back
        _sample("social17_s100_outputs", "rmat", n=1 << 17, ef=16, undirected=True, s=100, seed_counts=True,
                node_stats=True, signatures=True),
        # a million-node web graph, in the default form and with seed groups by reach
        _sample("rmat20_s256", "rmat", n=1 << 20, ef=16, s=256, device_seeds=True),
        _sample("rmat20_s256_reach", "rmat", n=1 << 20, ef=16, s=256, device_seeds=True, reach=True, signatures=True),
        # the largest graphs: rows far beyond the caches, both forms
        _sample("rmat24_s512", "rmat", n=1 << 24, ef=16, s=512, device_seeds=True, signatures=True),
        _sample("rmat24_s512_reach", "rmat", n=1 << 24, ef=16, s=512, device_seeds=True, reach=True),
        # long diameters: a lattice as a road network stands in for, hundreds
        # of rounds; and a small odd-sided one with few seeds
        _sample("grid4096_s128", "grid", side=4096, s=128, device_seeds=True),
        _sample("grid301_s9", "grid", side=301, s=9),
        # sixty-four uneven graphs measured in one call
        dict(name="batch64_s64", kind="batch", graphs=64, s=64),
        # ground truth of a small graph: every node a seed
        dict(name="exact13", kind="exact", n=1 << 13, ef=8, undirected=True, group=512),
        # memory-lean seeds, one bit per node
        dict(name="seq20_s256", kind="seq", n=1 << 20, ef=16, undirected=False, s=256),
        # a sample that grows until its error bound is met, on a graph just built
        dict(name="new_graph17_progressive", kind="new_graph", n=1 << 17, ef=16, undirected=False, group=256,
             pool=1536, target=1.0),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["rmat", "rmat", "rmat", "er", "grid", "batch", "exact", "seq", "new_graph"])
    und = rng.random() < 0.4
    if kind == "rmat":
        n = logint(1 << 12, 1 << 22)
        outs = n < (1 << 18) and rng.random() < 0.4
        return _sample(None, "rmat", n=n, ef=rng.randint(4, 24), undirected=und, s=logint(1, 512),
                       seed_counts=outs, node_stats=outs and rng.random() < 0.5, signatures=outs or rng.random() < 0.3,
                       device_seeds=rng.random() < 0.5, reach=not outs and rng.random() < 0.4)
    if kind == "er":
        n = logint(1000, 1 << 20)
        return _sample(None, "er", n=n, m=n * rng.randint(2, 12), undirected=und, s=logint(1, 512),
                       device_seeds=rng.random() < 0.5)
    if kind == "grid":
        return _sample(None, "grid", side=logint(40, 1500), s=logint(1, 200), device_seeds=rng.random() < 0.5)
    if kind == "batch":
        return dict(kind="batch", graphs=rng.randint(2, 64), s=logint(1, 64))
    if kind == "exact":
        return dict(kind="exact", n=logint(300, 1 << 13), ef=rng.randint(3, 12), undirected=und,
                    group=rng.choice([64, 200, 512]))
    if kind == "seq":
        return dict(kind="seq", n=logint(1 << 12, 1 << 20), ef=rng.randint(4, 16), undirected=und, s=logint(1, 256))
    return dict(kind="new_graph", n=logint(1 << 12, 1 << 18), ef=rng.randint(4, 16), undirected=und,
                group=rng.choice([64, 200, 256]), pool=logint(256, 1536), target=rng.choice([0.5, 1.0, 2.0]))


def _sample(name, graph, n=0, m=0, ef=0, side=0, undirected=False, s=64, device_seeds=False, reach=False,
            seed_counts=False, node_stats=False, signatures=False):
    case = dict(kind="sample", graph=graph, n=n, m=m, ef=ef, side=side, undirected=undirected or graph == "grid", s=s,
                device_seeds=device_seeds, reach=reach, seed_counts=seed_counts, node_stats=node_stats,
                signatures=signatures)
    return case if name is None else dict(name=name, **case)


# ------------------------------------------------------------------ inputs

def _rmat(n, ef, seed, device="cuda"):
    """R-MAT arcs (a, b, c, d = .57, .19, .19, .05) on n nodes: ids of the next
    power of two, scaled down to [0, n) when n is none."""
    gen = torch.Generator(device=device).manual_seed(seed)
    scale = max(1, (n - 1).bit_length())
    m = ef * n
    src = torch.zeros(m, dtype=torch.int64, device=device)
    dst = torch.zeros(m, dtype=torch.int64, device=device)
    for _ in range(scale):
        u = torch.rand(m, generator=gen, device=device)
        src.mul_(2).add_(u >= 0.76)
        dst.mul_(2).add_(((u >= 0.57) & (u < 0.76)) | (u >= 0.95))
    if n != 1 << scale:
        src.mul_(n).bitwise_right_shift_(scale)
        dst.mul_(n).bitwise_right_shift_(scale)
    return src.to(torch.int32), dst.to(torch.int32)


def _er(n, m, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ends = torch.randint(0, n, (2, m), generator=gen, device="cuda", dtype=torch.int32)
    return ends[0].contiguous(), ends[1].contiguous()


def _grid(side, seed):
    """side x side lattice, about a tenth of its edges deleted, and as many
    shortcuts per node as 1000 on 4096 x 4096 (at least one)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ids = torch.arange(side * side, dtype=torch.int32, device="cuda").view(side, side)
    a = torch.cat([ids[:, :-1].reshape(-1), ids[:-1].reshape(-1)])
    b = torch.cat([ids[:, 1:].reshape(-1), ids[1:].reshape(-1)])
    keep = torch.rand(a.numel(), generator=gen, device="cuda") >= 0.1
    cuts = torch.randint(0, side * side, (2, max(1, side * side * 1000 >> 24)), generator=gen, device="cuda",
                         dtype=torch.int32)
    return torch.cat([a[keep], cuts[0]]), torch.cat([b[keep], cuts[1]])


def _arcs(case, seed):
    if case.get("graph") == "er":
        return case["n"], *_er(case["n"], case["m"], seed)
    if case.get("graph") == "grid":
        return case["side"] ** 2, *_grid(case["side"], seed)
    return case["n"], *_rmat(case["n"], case["ef"], seed)


def _batch(graphs, s, seed):
    """The batched workload's mix: a third each of R-MATs (scales 10 to 16),
    lattices (sides 64 to 512) and paths (1000 to 20001 nodes)."""
    gs, third = [], max(1, graphs // 3)
    for k in range(graphs):
        q = k // 3
        if k % 3 == 0:
            gs.append(inputs.rmat(10 + q % 7, 8 + 4 * (q % 3), inputs.subseed(seed, 100 + k)))
        elif k % 3 == 1:
            side = 64 + (q * 448) // max(1, third - 1)
            gs.append(inputs.grid_graph(side, min(512, side)))
        else:
            gs.append(inputs.path_graph(1001 + (q * 19000) // max(1, third - 1)))
    seeds = [inputs.sample_seeds(g.n, s, inputs.subseed(seed, 200 + i)) for i, g in enumerate(gs)]
    return inputs.union_of(gs, seeds)


def _rounds(case):
    """Columns of the count tables the program keeps: enough for any seed's rounds."""
    if case["kind"] == "batch":
        return 20480
    return 8 * case["side"] + 64 if case.get("graph") == "grid" else 256


def _table(counts, rounds):
    """The counts in a table of fixed width, as a program that compares samples keeps them."""
    out = np.zeros(counts.shape[:-1] + (rounds,), counts.dtype)
    out[..., :counts.shape[-1]] = counts
    return out


def _seeds(n, s, seed):
    return inputs.sample_seeds(n, s, seed, distinct=s <= n // 2)


# ------------------------------------------------------------------ one pass

def prepare(case, seed):
    # device memory from PyTorch's caching allocator, as a program that also runs PyTorch sets it
    pp.use_torch_allocator(torch)
    kind = case["kind"]
    if kind == "batch":
        n, src, dst, offs, sd = _batch(case["graphs"], case["s"], seed)
        g = pp.pp_csr_build(n, src, dst, node_offsets=offs)
        run_ = pp.pp_seeds_init(g, sd, s=case["s"], opts=pp.options(persistent=True))
        return dict(kind=kind, case=case, graph=g, run=run_, seeds=sd)
    n, src, dst = _arcs(case, seed)
    torch.cuda.synchronize()
    if kind == "new_graph":
        return dict(kind=kind, case=case, n=n, src=src, dst=dst, pool=_seeds(n, case["pool"], seed))
    g = pp.pp_csr_build(n, src, dst, undirected=case["undirected"])
    if kind == "exact":
        return dict(kind=kind, case=case, graph=g, group=case["group"])
    sd = _seeds(n, case["s"], seed)
    if kind == "seq":
        return dict(kind=kind, case=case, graph=g, seeds=sd)
    opts = pp.options(seed_counts=case["seed_counts"], node_stats=case["node_stats"],
                      seed_groups=pp.PP_GROUPS_BY_REACH if case["reach"] else 0,
                      max_rounds=_rounds(case) - 1 if case["seed_counts"] else 0)
    run_ = pp.pp_seeds_init(g, sd, opts=opts)
    state = dict(kind=kind, case=case, graph=g, run=run_, seeds=sd)
    if case["device_seeds"]:
        state["seeds"] = torch.from_numpy(sd).cuda()
    if case["signatures"]:
        state["out"] = torch.empty(n, run_.words, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()
    return state


def run(state):
    kind, case = state["kind"], state["case"]
    rounds = _rounds(case)
    if kind in ("sample", "batch"):
        r = state["run"]
        pp.pp_seeds_reset(r, state["seeds"])
        counts, D = pp.pp_propagate_until_converged(r)
        out = [_table(counts, rounds), D]
        if case.get("seed_counts"):
            out.append(pp.pp_get_seed_counts(r, rounds))
        if case.get("node_stats"):
            out += list(pp.pp_get_node_stats(r))
        if case.get("signatures"):
            out.append(pp.pp_get_signatures(r, out=state["out"]))
        return out
    if kind == "exact":
        counts, D = pp.pp_exact_counts(state["graph"], state["group"], cap_rounds=rounds)
        return [_table(counts, rounds), D]
    if kind == "seq":
        counts, D, examined = pp.pp_propagate_s(state["graph"], state["seeds"], cap_rounds=rounds)
        return [_table(counts, rounds), D, examined]
    g = pp.pp_csr_build(state["n"], state["src"], state["dst"], undirected=case["undirected"])
    res = pp.pp_progressive_sample(g, state["pool"], case["group"], case["target"], 0.05, cap_rounds=rounds)
    g.free()
    res["counts"] = _table(res["counts"], rounds)
    return res


# ------------------------------------------------------------------ bounds

def work(case):
    """Each arc's column index once and each node's offset once, and each
    node's final row of s bits written once; a call with several groups of
    seeds writes each group's rows.  flops: one OR per arc and seed word,
    which every node needs at least once."""
    kind = case["kind"]
    if kind == "batch":
        third = case["graphs"] / 3.0
        n, m = third * (18e3 + 98e3 + 10.5e3), third * (220e3 + 390e3 + 21e3)
    elif case.get("graph") == "grid":
        n = case["side"] ** 2
        m = 3.6 * n
    else:
        n = case["n"]
        m = (case.get("m") or case["ef"] * n) * (2 if case["undirected"] else 1)
    seeds = {"exact": n, "new_graph": case.get("group")}.get(kind, case.get("s"))
    words = -(-seeds // 64)
    once = 4 * m + 8 * n
    if kind == "new_graph":   # the arcs in, both adjacencies out
        once += 8 * case["ef"] * n + 8 * m + 16 * n
    return {"bytes": int(once + 8 * words * n), "flops": int(m * words)}


def exact(case, seed):
    """The progressive sample's figures from a plain propagation in numpy; the
    other cases return whole numbers only."""
    if case["kind"] != "new_graph":
        return None
    n, src, dst = _arcs(case, seed)
    src, dst = src.cpu().numpy().astype(np.int64), dst.cpu().numpy().astype(np.int64)
    if case["undirected"]:
        src, dst = np.concatenate([src, dst]), np.concatenate([dst, src])
    key = np.unique((src * n + dst)[src != dst])
    src, dst = key // n, key % n
    pool = _seeds(n, case["pool"], seed)
    heads, first = np.unique(src, return_index=True)   # nodes with successors, and where their lists start
    total, used, groups, dmax = np.zeros(_rounds(case), np.int64), 0, 0, 0
    met, alpha, eps, bound = False, 0.0, 0.0, 0.0
    while used < len(pool) and not met:
        x = pool[used:used + case["group"]]
        sig = np.zeros((n, -(-len(x) // 64)), np.uint64)
        i = np.arange(len(x))
        np.bitwise_or.at(sig, (x, i >> 6), np.uint64(1) << (i & 63).astype(np.uint64))
        total[0] += len(x)
        for r in range(1, len(total)):
            if not len(heads):
                break
            new = np.bitwise_or.reduceat(sig[dst], first, axis=0) & ~sig[heads]
            got = int(np.unpackbits(new.view(np.uint8)).sum(dtype=np.int64))
            if got == 0:
                break
            sig[heads] |= new
            total[r] += got
            dmax = max(dmax, r)
        used, groups = used + len(x), groups + 1
        alpha = float(total.sum() - used) / (float(used) * (n - 1))
        eps = math.sqrt(math.log(2.0 / 0.05) / (2.0 * used))
        bound = 0.0 if dmax == 0 else (eps * dmax / alpha if alpha > 0 else math.inf)
        met = bound <= case["target"]
    return dict(seeds=used, groups=groups, met=met, D=dmax, alpha=alpha, eps=eps, bound=bound,
                counts=total)
