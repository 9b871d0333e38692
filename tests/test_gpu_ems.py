"""The mutual-selection baseline (Section II-C) on the GPU against the
oracle's weighted greedy: with fixed edge weights both reach the greedy
matching in descending weight order, so they must agree bit for bit."""
import time

import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2507_04420_amd as mm  # noqa: E402
from paper_2507_04420_amd import _lib  # noqa: E402


def to_dev(g):
    return torch.from_numpy(g.off).cuda(), torch.from_numpy(g.nbr).cuda()


GRAPHS = {
    "er": lambda: graphgen.er(30000, 10, seed=4),
    "er_int32": lambda: graphgen.er(65536, 16, seed=1).with_int32_offsets(),
    "rmat": lambda: graphgen.rmat(16, seed=2),
    "grid": lambda: graphgen.grid(120, 97),
    "clique": lambda: graphgen.from_edges(64, [(i, j) for i in range(64) for j in range(i + 1, 64)]),
    "star": lambda: graphgen.from_edges(5001, [(0, j) for j in range(1, 5001)]),
    "loops_dups": lambda: graphgen.from_edges(
        50, [(i, (i * 7) % 50) for i in range(50)] * 2 + [(3, 3), (9, 9)], dedup=False, sort=False),
    "empty": lambda: graphgen.from_edges(9, np.zeros((0, 2))),
}


@pytest.mark.parametrize("name", sorted(GRAPHS))
@pytest.mark.parametrize("seed", [1, 77])
def test_ems_equals_weighted_greedy(name, seed):
    g = GRAPHS[name]()
    off, nbr = to_dev(g)
    h = mm.Graph(off, nbr, symmetric=True)
    mate, st = h.ems(seed=seed)
    got = mate.cpu().numpy()
    want, pairs = oracle.greedy_weighted(g, seed)
    np.testing.assert_array_equal(got, want)
    assert st["pairs"] == pairs
    assert oracle.check(g, got).ok
    assert st["iterations"] >= 1
    if g.m:
        assert st["touched"] >= g.m  # the first selection scans every list


def test_ems_needs_symmetric_handle():
    g = graphgen.er(100, 4, seed=1)
    off, nbr = to_dev(g)
    h = mm.Graph(off, nbr)
    with pytest.raises(mm.MMError) as ei:
        h.ems()
    assert ei.value.status == _lib.MM_ERR_UNSUPPORTED


def test_ems_reads_more_than_skipper():
    # the contrast of Section II-C: several full passes against one early-exit pass
    g = graphgen.rmat(18, seed=3)
    off, nbr = to_dev(g)
    h = mm.Graph(off, nbr, symmetric=True, stats=True)
    out = h.run()
    h.sync()
    skipper = h.stats()
    _, st = h.ems(seed=5)
    assert oracle.check(g, out.cpu().numpy()).ok
    assert st["iterations"] >= 2
    assert st["touched"] > 2 * (skipper["touched"] + skipper["assist_reads"])


def _mix(z):
    z = z + np.uint64(0x9E3779B97F4A7C15)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def rounds(csr, seed):
    """(iterations, ids read) of the mutual selection, round by round: the last
    round finds nothing to select; a round reads the lists of free vertices."""
    off = csr.off.astype(np.int64)
    deg = np.diff(off)
    x, y = np.repeat(np.arange(csr.n), deg), csr.nbr.astype(np.int64)
    key = (np.minimum(x, y).astype(np.uint64) << np.uint64(32)) | np.maximum(x, y).astype(np.uint64)
    with np.errstate(over="ignore"):
        w = _mix(_mix(np.array([seed], dtype=np.uint64)) ^ key)
    order = np.lexsort((key, ~w, x))  # each list by falling weight, then rising key
    x, y = x[order], y[order]
    mate = np.full(csr.n, -1)
    iterations = touched = 0
    while True:
        free = mate == -1
        iterations += 1
        touched += int(deg[free].sum())
        live = np.flatnonzero(free[x] & free[y] & (x != y))
        if live.size == 0:
            return iterations, touched
        first = live[np.r_[True, x[live][1:] != x[live][:-1]]]
        sel = np.full(csr.n, -1)
        sel[x[first]] = y[first]
        v = np.flatnonzero(sel >= 0)
        m = v[sel[sel[v]] == v]
        mate[m] = sel[m]


def _clique(n, among=0):
    return graphgen.from_edges(max(n, among), [(i, j) for i in range(n) for j in range(i + 1, n)])


# runs of 1 to 12 iterations: the counters are read back for eight iterations at
# a time, or (few entries) for one or two first, and a run may end before, at and
# after such a wait
@pytest.mark.parametrize("make,seed,iterations", [
    (lambda: graphgen.from_edges(9, np.zeros((0, 2))), 1, 1),
    (lambda: graphgen.from_edges(9, [(4, 4)]), 1, 1),
    (lambda: graphgen.from_edges(10, [(i, i + 1) for i in range(9)]), 3, 2),
    (lambda: graphgen.from_edges(500, [(2 * i, 2 * i + 1) for i in range(250)]), 1, 2),
    (lambda: graphgen.grid(4, 4), 1, 3),
    (lambda: graphgen.from_edges(40, [(i, i + 1) for i in range(9)]), 1, 3),
    (lambda: graphgen.from_edges(100000, [(i, i + 1) for i in range(30000)]), 1, 5),
    (lambda: _clique(300, 100000), 1, 9),
    (lambda: _clique(300, 100000), 2, 10),
    (lambda: _clique(300, 100000), 6, 11),
    (lambda: graphgen.er(10, 8, seed=4), 1, 4),
    (lambda: graphgen.er(300, 8, seed=4), 3, 7),
    (lambda: graphgen.er(1000, 8, seed=4), 4, 8),
    (lambda: _clique(400), 9, 9),
    (lambda: graphgen.er(30000, 8, seed=4), 3, 10),
    (lambda: _clique(400), 1, 10),
    (lambda: _clique(400), 3, 11),
    (lambda: _clique(400), 7, 12),
])
def test_ems_counts_every_iteration(make, seed, iterations):
    csr = make()
    want = rounds(csr, seed)
    assert want[0] == iterations
    h = mm.Graph(*to_dev(csr), symmetric=True)
    mate, st = h.ems(seed=seed)
    np.testing.assert_array_equal(mate.cpu().numpy(), oracle.greedy_weighted(csr, seed)[0])
    assert (st["iterations"], st["touched"]) == want
    h.close()


def test_ems_short_run_pays_for_its_own_iterations():
    # an edgeless graph (one iteration) against one of eight; with eight
    # iterations launched for either it took 0.9 of the time, with its own 0.4
    def median(csr):
        h = mm.Graph(*to_dev(csr), symmetric=True)
        h.ems(seed=4)
        times = []
        for _ in range(21):
            torch.cuda.synchronize()
            t = time.perf_counter()
            h.ems(seed=4)
            times.append(time.perf_counter() - t)
        h.close()
        return 1e6 * sorted(times)[10]

    one = median(graphgen.from_edges(1000, np.zeros((0, 2))))
    eight = median(graphgen.er(1000, 8, seed=4))
    print("%.0f us for one iteration, %.0f us for eight" % (one, eight))
    assert one < 0.65 * eight
