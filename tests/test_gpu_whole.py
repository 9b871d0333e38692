"""Graphs that one wavefront sweeps with their states in LDS: the loop of their
own that the plain build runs has the schedule of the general sweep, which the
instrumented build runs, so the two give the same mates, entry by entry, and
the counters of the one describe the other."""
import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2507_04420_amd as mm  # noqa: E402

TUNINGS = {
    "default": {},
    "serving": dict(upper_only=1, probe_first=1, wait_release=1),
    "one_candidate": dict(probe_first=2, scan_width=3, wait_release=1),
    "narrow": dict(scan_width=1, assist_after=1),
    "assist": dict(assist_after=2, upper_only=1, scan_width=2),
    "ordered": dict(order_lists=2, upper_only=1, probe_first=1, assist_after=4),
    "ordered1": dict(order_lists=1, scan_width=4, assist_after=16),
}


def shuffled(n, m, seed):
    """A multigraph with loops and repeated entries, lists in no order."""
    rng = np.random.default_rng(seed)
    a, b = rng.integers(0, n, m), rng.integers(0, max(1, n // 7), m)
    e = np.stack([a, b], 1)
    return graphgen.from_edges(n, e, symmetric=True, dedup=False, sort=False)


def star(n):
    return graphgen.from_edges(n, [(0, v) for v in range(1, n)] + [(n - 1, v) for v in range(1, n - 1)])


# a source per lane and the next (64), chunks of the queue (128), the first and
# last ids of a graph (fewer than four entries in all), the largest graphs
GRAPHS = {
    "none1": lambda: graphgen.from_edges(1, np.zeros((0, 2), dtype=np.int64)),
    "edge2": lambda: graphgen.from_edges(2, [(0, 1)]),
    "path3": lambda: graphgen.from_edges(3, [(0, 1), (1, 2)]),
    "one_edge200": lambda: graphgen.from_edges(200, [(198, 199)]),
    "er63": lambda: graphgen.er(63, 3.0, seed=1),
    "er64": lambda: graphgen.er(64, 5.0, seed=2),
    "er65": lambda: graphgen.er(65, 8.0, seed=3),
    "er129": lambda: graphgen.er(129, 30.0, seed=4),
    "multi777": lambda: shuffled(777, 4000, 5),
    "star700": lambda: star(700),
    "star16384": lambda: star(16384),
    "er5003": lambda: graphgen.er(5003, 12.0, seed=6),
    "grid128": lambda: graphgen.grid(128, 128),
    "grid127x129": lambda: graphgen.grid(127, 129),
    "er16383": lambda: graphgen.er(16383, 17.0, seed=7),
    "rmat14": lambda: graphgen.rmat(14, 16, seed=8),
}


@pytest.mark.parametrize("gname", sorted(GRAPHS))
def test_whole_loop_has_the_sweeps_schedule(gname):
    csr = GRAPHS[gname]()
    for tname, over in TUNINGS.items():
        for c in (csr, csr.with_int32_offsets()):
            off, nbr = torch.from_numpy(c.off).cuda(), torch.from_numpy(c.nbr).cuda()
            got = []
            for stats in (False, True):
                t = mm.Tuning.default()
                for k, v in over.items():
                    setattr(t, k, v)
                g = mm.Graph(off, nbr, symmetric=True, stats=stats, tuning=t)
                got.append(g.run().cpu().numpy())
                g.sync()
                if stats:
                    assert g.stats()["pairs"] * 2 == int((got[1] >= 0).sum()), (gname, tname)
                g.close()
            assert np.array_equal(got[0], got[1]), (gname, tname, int((got[0] != got[1]).sum()))
            assert oracle.check(c, got[0]).ok, (gname, tname)


# a batch gives each of them the same mates, in whatever order it runs them
def test_whole_batch_same_as_alone():
    parts = [GRAPHS[k]() for k in sorted(GRAPHS)]
    graphs = [(torch.from_numpy(p.off).cuda(), torch.from_numpy(p.nbr).cuda()) for p in parts]
    b = mm.Batch.from_list(graphs, symmetric=True)
    out = b.run().cpu().numpy()
    b.sync()
    for g, p in enumerate(parts):
        h = mm.Graph(*graphs[g], symmetric=True)
        alone = h.run().cpu().numpy()
        h.close()
        assert np.array_equal(out[b.vtx_off[g]:b.vtx_off[g + 1]], alone), g
    b.close()


# the loop-trip budget ends it with the error flag and no vertex half matched
def test_whole_loop_budget():
    csr = graphgen.er(5000, 9.0, seed=9)
    t = mm.Tuning.default()
    t.iter_cap = 40
    g = mm.Graph(torch.from_numpy(csr.off).cuda(), torch.from_numpy(csr.nbr).cuda(), symmetric=True, tuning=t)
    mate = g.run()
    with pytest.raises(mm.MMError):
        g.sync()
    mate = mate.cpu().numpy()
    v = np.flatnonzero(mate >= 0)
    assert len(v) and np.array_equal(mate[mate[v]], v)
    g.close()
