"""The pair list (mm_pairs) at the sizes where its tiles of vertices begin, end
and grow, on matchings made on the CPU."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2507_04420_amd as mm  # noqa: E402


# the edges of a tile of vertices, and of the sizes at which tiles grow
@pytest.mark.parametrize("n", [1, 2, 63, 65, 255, 256, 257, 2047, 2049, 65535, 65536, 65537, 131073,
                               (1 << 21) - 1, 1 << 21, (1 << 21) + 8191, (1 << 24) + 3])
def test_pairs_tile_edges(n):
    rng = np.random.default_rng(n)
    ids = rng.permutation(n).astype(np.int32)
    k = int(n * 0.4)
    mate = np.full(n, -1, dtype=np.int32)
    mate[ids[:k]], mate[ids[k:2 * k]] = ids[k:2 * k], ids[:k]
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    g = mm.Graph(off, torch.zeros(0, dtype=torch.int32, device="cuda"))
    got = g.pairs(torch.from_numpy(mate).cuda()).cpu().numpy()
    g.close()
    assert got.shape == (k, 2)
    got = got[np.argsort(got[:, 0])]
    lower = np.flatnonzero(mate > np.arange(n))
    assert np.array_equal(got[:, 0], lower) and np.array_equal(got[:, 1], mate[lower])
