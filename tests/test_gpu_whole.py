"""Graphs that one wavefront sweeps with their states in LDS: the loop of their
own that the plain build runs has the schedule of the general sweep, which the
instrumented build runs, so the two give the same mates, entry by entry, and
the counters of the one describe the other."""
import hashlib

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


# one wavefront with its states in device memory: the matching is that of the
# schedule alone, so what several wavefronts share a sweep by (noted sources,
# the guess on a shared word) must leave it as it was
WHOLE_PINS = {
    ("er5003", "u8_cas"): "dd7c835c81fbf2d4",
    ("er5003", "u2_two"): "74e44f21c5cc2317",
    ("er5003", "u32_cas"): "d5fd7bd0aa5263e2",
    ("er5003", "u8_hint_upper"): "02edf171caa199b4",
    ("er5003", "u8_relabel"): "8446d6584d0716b5",
    ("grid127x129", "u8_cas"): "31059041ea52c699",
    ("grid127x129", "u2_two"): "baee8bc2dda2f152",
    ("grid127x129", "u32_cas"): "baee8bc2dda2f152",
    ("grid127x129", "u8_hint_upper"): "31f3839783ed7d29",
    ("grid127x129", "u8_relabel"): "57ab1fefec1eb504",
    ("rmat13", "u8_cas"): "07c26d0e6f7e62a5",
    ("rmat13", "u2_two"): "10015fd4b129255e",
    ("rmat13", "u32_cas"): "3735ae67668a33b9",
    ("rmat13", "u8_hint_upper"): "4ed7934b9f9b8027",
    ("rmat13", "u8_relabel"): "d7539135304c8648",
}
WHOLE_TUNINGS = {
    "u8_cas": dict(layout=0),
    "u2_two": dict(layout=2, protocol=1),
    "u32_cas": dict(),
    "u8_hint_upper": dict(layout=0, hint=2, upper_only=1, wait_release=1),
    "u8_relabel": dict(layout=0, relabel=1),
}
WHOLE_GRAPHS = {
    "er5003": lambda: graphgen.er(5003, 12.0, seed=6),
    "grid127x129": lambda: graphgen.grid(127, 129),
    "rmat13": lambda: graphgen.rmat(13, 8, seed=8),
}


@pytest.mark.parametrize("graph,tuning", list(WHOLE_PINS))
def test_whole_in_device_memory_keeps_its_schedule(graph, tuning):
    g = WHOLE_GRAPHS[graph]()
    t = mm.Tuning.default()
    t.whole_graph_lds = 0
    for k, v in WHOLE_TUNINGS[tuning].items():
        setattr(t, k, v)
    h = mm.Graph(torch.from_numpy(g.off).cuda(), torch.from_numpy(g.nbr).cuda(),
                 symmetric=True, tuning=t)
    for _ in range(2):
        mate = h.run().cpu().numpy()
        assert hashlib.sha1(mate.tobytes()).hexdigest()[:16] == WHOLE_PINS[graph, tuning]
    h.sync()
    h.close()


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1000, 16384])
@pytest.mark.parametrize("dtype", [torch.int32, torch.int64])
def test_graph_without_entries(n, dtype):
    # nothing to sweep: every vertex unmatched, alone and between other members
    off = torch.zeros(n + 1, dtype=dtype, device="cuda")
    nbr = torch.zeros(0, dtype=torch.int32, device="cuda")
    out = torch.full((n,), -5, dtype=torch.int32, device="cuda")
    g = mm.Graph(off, nbr, symmetric=True)
    g.run(out)
    g.sync()
    assert (out == -1).all()
    g.close()
    pair = (torch.tensor([0, 1, 2], device="cuda"), torch.tensor([1, 0], dtype=torch.int32, device="cuda"))
    b = mm.Batch.from_list([pair, (off.long(), nbr), pair, (off.long(), nbr)], symmetric=True)
    out = torch.full((b.N,), -5, dtype=torch.int32, device="cuda")
    b.run(out)
    b.sync()
    assert out.tolist() == ([1, 0] + [-1] * n) * 2
    b.close()
