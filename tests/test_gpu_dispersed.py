"""Sweeps whose lanes are dispersed (tuning.disperse) by several wavefronts,
which note in LDS the sources they match themselves, one bit for each of the
first 4096 of a block, and pass over a queued source so noted. Checked where a
wrong bit would lose a source: blocks longer than the bits, pieces of long
lists, relabelled graphs, outputs written by the sweep itself, one-sided lists.
The graphs are local ones (meshes, paths), on which sources are passed over."""
import numpy as np
import pytest

import graphgen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2507_04420_amd as mm  # noqa: E402
from paper_2507_04420_amd import _lib  # noqa: E402

U8, U32, U2 = _lib.MM_LAYOUT_U8, _lib.MM_LAYOUT_U32, _lib.MM_LAYOUT_U2
TWO = _lib.MM_PROTOCOL_TWO_PHASE


def tuning(**kw):
    return mm.Tuning(**dict(dict(disperse=1, whole_graph_vertices=0), **kw))


TUNINGS = {
    "u8_lazy_64": tuning(layout=U8, lazy_init=1, wave_vertices=64),
    "u8_64_wg64": tuning(layout=U8, wave_vertices=64, wg_size=64),
    "u8_256_wg192": tuning(layout=U8, wave_vertices=256, wg_size=192),
    "u32_256_release": tuning(wave_vertices=256, wait_release=1),
    "u32_upper_release": tuning(wave_vertices=256, wait_release=1, upper_only=1, probe_first=1),
    "u2_two_hint_lazy": tuning(layout=U2, protocol=TWO, hint=1, lazy_init=1, wave_vertices=512),
    # blocks of twice the bits, and one source beyond them
    "u2_8192": tuning(layout=U2, wave_vertices=8192, min_waves=0),
    "u32_two_8192": tuning(protocol=TWO, wave_vertices=8192, min_waves=0),
    "u8_4160_bytehint": tuning(layout=U8, wave_vertices=4160, min_waves=0, hint=2),
    # long lists in pieces, each swept by a lane, beside dispersed blocks
    "u32_pieces": tuning(hub_wave=0, hub_degree=4, hub_chunk=3),
    "u8_pieces_1": tuning(layout=U8, hub_wave=0, hub_degree=1, hub_chunk=1, wave_vertices=128),
    "u32_pieces_wave": tuning(hub_wave=1, hub_degree=2, hub_chunk=2, wg_size=128),
    "u8_relabel": tuning(layout=U8, relabel=1, wave_vertices=256),
    "u32_relabel2": tuning(relabel=2, hot_degree=3, wave_vertices=8192, min_waves=0),
}


def wheel(n):  # a path whose vertices all join one hub in its middle
    return graphgen.from_edges(n, [(i, i + 1) for i in range(n - 1)] + [(n // 2, i) for i in range(0, n, 3)])


GRAPHS = {
    "mesh": lambda: graphgen.grid(107, 97),
    "path": lambda: graphgen.from_edges(9001, [(i, i + 1) for i in range(9000)]),
    "wheel": lambda: wheel(9000),
    "er": lambda: graphgen.er(10007, 5, seed=4),
    "one_sided_mesh": lambda: graphgen.from_edges(
        9000, [(i, i + 1) for i in range(8999) if i % 90 != 89] + [(i, i + 90) for i in range(8910)],
        symmetric=False),
    "one_sided_down": lambda: graphgen.from_edges(8500, [(i + 1, i) for i in range(8499)], symmetric=False),
}


@pytest.mark.parametrize("gname", sorted(GRAPHS))
@pytest.mark.parametrize("tname", sorted(TUNINGS))
def test_dispersed_sweep_loses_no_source(gname, tname):
    t = TUNINGS[tname]
    csr = GRAPHS[gname]()
    sym = not gname.startswith("one_sided")
    for k, stats in enumerate((False, False, True)):
        c = csr.with_int32_offsets() if k == 1 else csr
        g = mm.Graph(torch.from_numpy(c.off).cuda(), torch.from_numpy(c.nbr).cuda(), symmetric=sym, tuning=t,
                     stats=stats)
        out = torch.empty(csr.n, dtype=torch.int32, device="cuda")
        for _ in range(3):
            out.fill_(-5)  # what a lost source would leave in a lazy output
            g.run(out)
            g.sync()
            got = oracle.check(csr, out.cpu().numpy())
            assert got.ok, (gname, tname, got)
        if stats:
            assert 3 * got.size * 0.9 < g.stats()["pairs"] < 3 * got.size * 1.1
        g.close()


@pytest.mark.parametrize("tname", ["u8_lazy_64", "u8_256_wg192", "u32_256_release", "u2_8192", "u32_pieces",
                                   "u2_two_hint_lazy"])
@pytest.mark.parametrize("mesh", [0, 64, 8192])
def test_dispersed_batch_loses_no_source(tname, mesh):
    t = mm.Tuning(**dict(TUNINGS[tname].as_dict(), mesh_wave_vertices=mesh, disperse=int(mesh == 0)))
    parts = [GRAPHS[k]() for k in ("mesh", "er", "path", "wheel")] + [graphgen.grid(3, 2)]
    b = mm.Batch.from_list([(torch.from_numpy(p.off).cuda(), torch.from_numpy(p.nbr).cuda()) for p in parts],
                           symmetric=True, tuning=t)
    out = torch.empty(b.N, dtype=torch.int32, device="cuda")
    for _ in range(3):
        out.fill_(-5)
        b.run(out)
        b.sync()
        mate = out.cpu().numpy()
        for g, p in enumerate(parts):
            assert oracle.check(p, mate[b.vtx_off[g]:b.vtx_off[g + 1]]).ok, (tname, mesh, g)
    b.close()
