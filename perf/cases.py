"""The work a user of this library has it do, as timed cases.

Every case is one pass through the public entry points (``maximal_matching``,
``Graph``, ``Batch``, their ``check``, ``pairs`` and ``ems``), over the graph
families this repository generates for its tests and its benchmark: sparse
random graphs (ER), skewed ones (R-MAT, 0.57/0.19/0.19/0.05, permuted ids) and
4-neighbour meshes. A mesh here lacks a fiftieth of its links, drawn from the
seed, so that two seeds give two graphs.

What a pass returns. A graph that one wavefront sweeps (at most 16384
vertices) has one result, and the pass returns its mates. On a larger graph
the lanes race and several maximal matchings are right (two passes over the
same graph differ in a fiftieth to a third of their mates), so such a pass is
the one the quick start, the autotuner and the benchmark take: run, sync, then
the device check, whose verdict it returns: every count of violations, and the
entries the pass covered. (The count of matched vertices is left out: it
varies with the matching.)
"""
import math
import random

import torch

import paper_2507_04420_amd as mm
from paper_2507_04420_amd import autotune, serve

WHOLE = 16384  # the largest graph one wavefront sweeps by default
VIOLATIONS = ("out_of_range", "self_mate", "asymmetric", "not_edge", "uncovered")


def listed():
    return [
        # the smallest call: a script that matches one little graph, create and wait included
        dict(name="one_shot_er1k", do="one_shot", family="er", n=1000, degree=8.0, symmetric=True, wide=True),
        # a small skewed graph matched again and again through one handle
        dict(name="whole_rmat13", do="whole", family="rmat", n=1 << 13, degree=16.0, symmetric=True, wide=True),
        # the same for a CSR that holds each edge once, with int32 offsets
        dict(name="whole_one_sided_5003", do="whole", family="er", n=5003, degree=12.0, symmetric=False, wide=False),
        # serving: the small requests that are waiting become one list batch, created for this one launch
        dict(name="serve_48_small", do="serve", members=48, least=1000, most=WHOLE, spec=1),
        # offline: many small graphs in one handle, replayed as a graph
        dict(name="batch_1024_small", do="batch", members=1024, least=1000, most=WHOLE, spec=2),
        # the batch workload's mixture (1e3 to 2e5 vertices) with its tuned entry
        dict(name="batch_256_mix", do="batch_mix", members=256, least=1000, most=200000, spec=3),
        # the benchmark's latency leg: int32 offsets
        dict(name="er_65536", do="verified", family="er", n=65536, degree=16.0, symmetric=True, wide=False),
        # a large job of the serving workload: it makes its own handle and runs once
        dict(name="solo_rmat18", do="solo", family="rmat", n=1 << 18, degree=16.0, symmetric=True, wide=True),
        # a large random graph, its lists reordered once when the handle is made
        dict(name="er_4m", do="verified", family="er", n=4000037, degree=16.0, symmetric=True, wide=True),
        # a mesh of ten million vertices, as the serving workload's large meshes
        dict(name="mesh_3168", do="verified", family="mesh", n=3168 * 3168, degree=4.0, symmetric=True, wide=True),
        # the headline's family and tuned entry (R-MAT from 2^25 vertices on)
        dict(name="rmat25", do="verified", family="rmat", n=1 << 25, degree=32.0, symmetric=True, wide=True),
        # what a multilevel coarsening does with a matching: list the pairs, map each vertex to its coarse one
        dict(name="coarsen_8m", do="coarsen", n=8000009, matched=0.8),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    do = rng.choice(("one_shot", "whole", "whole", "serve", "batch", "batch_mix", "verified", "verified",
                     "verified", "solo", "coarsen", "weighted"))
    if do == "serve":
        return dict(do=do, members=_log(rng, 1, 200), least=_log(rng, 64, 4000), most=WHOLE, spec=rng.randrange(1 << 20))
    if do == "batch":
        return dict(do=do, members=_log(rng, 16, 2000), least=_log(rng, 64, 4000), most=WHOLE, spec=rng.randrange(1 << 20))
    if do == "batch_mix":
        return dict(do=do, members=_log(rng, 16, 300), least=1000, most=200000, spec=rng.randrange(1 << 20))
    if do == "coarsen":
        return dict(do=do, n=_log(rng, 1000, 8000000), matched=rng.choice((0.1, 0.5, 0.8, 1.0)))
    family = rng.choice(("er", "rmat", "mesh"))
    lo, hi = {"one_shot": (64, WHOLE), "whole": (64, WHOLE), "solo": (WHOLE + 1, 1 << 21),
              "weighted": (1000, 1 << 19), "verified": (WHOLE + 1, 1 << 23)}[do]
    n = _log(rng, lo, hi)
    if family == "rmat":
        n = 1 << min(max(int(round(math.log2(n))), 6 if lo < WHOLE else 15), int(math.log2(hi)))
    degree = {"er": rng.uniform(4.0, 32.0), "rmat": rng.choice((16.0, 32.0)), "mesh": 4.0}[family]
    return dict(do=do, family=family, n=n, degree=degree, symmetric=do in ("solo", "verified", "weighted") or rng.random() < 0.7,
                wide=rng.random() < 0.7)


# ------------------------------------------------------------------ inputs

def _csr(n, a, b, symmetric):
    """Sorted lists without loops and without duplicates: (int64 offsets, int32 ids)."""
    keep = a != b
    a, b = a[keep], b[keep]
    key = torch.cat([a * n + b, b * n + a]) if symmetric else torch.minimum(a, b) * n + torch.maximum(a, b)
    key = torch.unique(key)
    src = torch.div(key, n, rounding_mode="floor")
    off = torch.zeros(n + 1, dtype=torch.int64, device=key.device)
    torch.cumsum(torch.bincount(src, minlength=n), 0, out=off[1:])
    return off, (key - src * n).to(torch.int32)


def _ends(family, n, degree, g):
    """The two ends of each drawn link of one graph."""
    dev = g.device
    if family == "mesh":
        w = max(1, math.isqrt(n))
        i = torch.arange(n, device=dev)
        right, down = i[(i % w != w - 1) & (i + 1 < n)], i[i + w < n]
        a, b = torch.cat([right, down]), torch.cat([right + 1, down + w])
        keep = torch.rand(a.numel(), generator=g, device=dev) >= 0.02
        return a[keep], b[keep]
    m = int(n * degree / 2)
    if family == "er":
        return (torch.randint(n, (m,), generator=g, device=dev), torch.randint(n, (m,), generator=g, device=dev))
    a = torch.zeros(m, dtype=torch.int64, device=dev)
    b = torch.zeros_like(a)
    for _ in range(n.bit_length() - 1):
        r = torch.rand(m, generator=g, device=dev)
        a.mul_(2).add_(r >= 0.76)
        b.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    ids = torch.randperm(n, generator=g, device=dev)
    return ids[a], ids[b]


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _graph(case, seed):
    n = case["n"]
    off, nbr = _csr(n, *_ends(case["family"], n, case["degree"], _generator(seed)), case.get("symmetric", True))
    return (off if case.get("wide", True) else off.to(torch.int32)), nbr


def _members(case):
    """(family, vertices, degree) of each member, the mixture's recipe."""
    rng = random.Random(case["spec"])
    got = []
    for _ in range(case["members"]):
        family, n = rng.choice(("er", "mesh", "rmat")), _log(rng, case["least"], case["most"])
        if family == "rmat":
            n = 1 << min(int(math.log2(case["most"])), max(6, int(round(math.log2(n)))))
        got.append((family, n, {"er": rng.uniform(4.0, 32.0), "mesh": 4.0, "rmat": 16.0}[family]))
    return got


def _concat(case, seed):
    """All members in one CSR of global positions and local ids, and the host's vertex offsets."""
    g = _generator(seed)
    specs = _members(case)
    vtx = [0]
    ends = []
    for family, n, degree in specs:
        a, b = _ends(family, n, degree, g)
        ends.append((a + vtx[-1], b + vtx[-1]))
        vtx.append(vtx[-1] + n)
    off, nbr = _csr(vtx[-1], torch.cat([e[0] for e in ends]), torch.cat([e[1] for e in ends]), True)
    first = torch.repeat_interleave(torch.tensor(vtx[:-1], device="cuda"), off[torch.tensor(vtx[1:], device="cuda")]
                                    - off[torch.tensor(vtx[:-1], device="cuda")])
    return off, (nbr - first).to(torch.int32), vtx


def prepare(case, seed):
    do = case["do"]
    if do in ("serve", "batch", "batch_mix"):
        off, nbr, vtx = _concat(case, seed)
        if do == "serve":
            cut = off[torch.tensor(vtx, device="cuda")].tolist()
            graphs = [((off[v:w + 1] - e).contiguous(), nbr[e:f].clone())
                      for v, w, e, f in zip(vtx, vtx[1:], cut, cut[1:])]
            return dict(do=do, graphs=graphs, tuning=serve.batch_tuning())
        b = mm.Batch(off, nbr, vtx, symmetric=True, capture=True,
                     tuning=autotune.tuned("batch") if do == "batch_mix" else None)
        return dict(do=do, batch=b, out=torch.empty(b.N, dtype=torch.int32, device="cuda"))
    if do == "coarsen":  # a given matching of n vertices; the handle's graph holds its edges
        n, g = case["n"], _generator(seed)
        ids = torch.randperm(n, generator=g, device="cuda")
        k = int(n * case["matched"] / 2)
        off, nbr = _csr(n, ids[:k], ids[k:2 * k], True)
        mate = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        mate[ids[:k]], mate[ids[k:2 * k]] = ids[k:2 * k].to(torch.int32), ids[:k].to(torch.int32)
        return dict(do=do, graph=mm.Graph(off, nbr, symmetric=True), mate=mate)
    off, nbr = _graph(case, seed)
    state = dict(do=do, off=off, nbr=nbr, symmetric=case["symmetric"])
    if do == "solo":
        state["tuning"] = serve.solo_tuning(off.cpu().numpy())
    elif do == "verified":
        t = autotune.tuned(autotune.classify(off.cpu().numpy()))
        state["graph"] = mm.Graph(off, nbr, symmetric=True, tuning=t)
    elif do in ("whole", "weighted"):
        state["graph"] = mm.Graph(off, nbr, symmetric=case["symmetric"])
    if do != "one_shot":
        state["out"] = torch.empty(case["n"], dtype=torch.int32, device="cuda")
    return state


# ------------------------------------------------------------------ passes

def _verdict(h, mate, entries):
    h.sync()
    c = h.check(mate)
    return dict({f: c[f] for f in VIOLATIONS}, ok=c["ok"], entries=entries)


def run(state):
    do = state["do"]
    if do == "one_shot":
        return mm.maximal_matching(state["off"], state["nbr"], symmetric=state["symmetric"])
    if do == "whole":
        return state["graph"].run(state["out"])
    if do == "verified":
        g = state["graph"]
        return _verdict(g, g.run(state["out"]), g.m)
    if do == "solo":
        g = mm.Graph(state["off"], state["nbr"], symmetric=True, tuning=state["tuning"])
        verdict = _verdict(g, g.run(state["out"]), g.m)
        g.close()
        return verdict
    if do == "serve":
        b = mm.Batch.from_list(state["graphs"], symmetric=True, tuning=state["tuning"])
        mate = b.run()
        b.sync()
        b.close()
        return mate
    if do == "batch":
        return state["batch"].run(state["out"])
    if do == "batch_mix":
        b = state["batch"]
        return _verdict(b, b.run(state["out"]), b.neighbors.numel())
    if do == "weighted":
        return state["graph"].ems(1, state["out"])[0]
    # coarsen: the pairs' order is not specified, the map made from them does not depend on it
    g = state["graph"]
    pairs = g.pairs(state["mate"])
    coarse = torch.arange(g.n, dtype=torch.int32, device="cuda")
    coarse[pairs[:, 1].long()] = pairs[:, 0]
    return coarse


def work(case):
    """The offsets once, at least two ids of each vertex (what a sequential pass with early exit reads on a sparse graph is more), and the
    mates once; with a verdict the mates are read again. Listing pairs reads the mates and writes the pairs and the map."""
    do = case["do"]
    if do == "coarsen":
        return dict(bytes=4.0 * case["n"] * (2 + case["matched"]), flops=0)
    specs = _members(case) if do in ("serve", "batch", "batch_mix") else [(case["family"], case["n"], case["degree"])]
    wide = 8 if case.get("wide", True) else 4
    verdict = 4 if do in ("verified", "solo", "batch_mix") else 0
    return dict(bytes=float(sum(n * (wide + 4 * min(2.0, d) + 4 + verdict) for _, n, d in specs)), flops=0)


def exact(case, seed):
    """Mates, maps and counts are whole numbers: none is a rounded value."""
    return None
