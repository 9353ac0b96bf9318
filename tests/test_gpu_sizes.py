"""Cluster lists (roots ascending, sizes) against the CPU oracle where the way
they are placed can go wrong: one tile column and more than 64 of them, rows
that end a tile early, and a little below and above the number of row counts up
to which the tiles add up the counts themselves (whole numbers: equal)."""
import numpy as np
import pytest

import oracle
import paper_1105_5804_amd as sw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("W,H,tile_h", [
    (1, 1, 0), (100, 1500, 0), (129, 64, 16), (300, 131, 32), (8500, 70, 0), (8323, 200, 128), (2000, 1024, 0),
    (2048, 1025, 0), (4100, 700, 0),
])
@pytest.mark.parametrize("mode", ["sites_open", "bonds_periodic"])
def test_roots_and_sizes(W, H, tile_h, mode):
    g = np.random.default_rng(W * 10007 + H)
    inp = (g.random((H, W)) < 0.6).astype(np.uint8) if mode == "sites_open" else g.integers(0, 4, (H, W), dtype=np.uint8)
    labels, roots, sizes, n = sw.ccl_label(torch.from_numpy(inp).cuda(), mode, sizes=True, tile_h=tile_h)
    flat = inp.reshape(-1)
    want, _ = oracle.label_sites(W, H, flat) if mode == "sites_open" else oracle.label_bonds(W, H, flat)
    lab = labels.cpu().numpy().reshape(-1)
    assert np.array_equal(lab, want)
    r, c = np.unique(lab[lab >= 0], return_counts=True)
    assert n == len(r)
    assert np.array_equal(roots.cpu().numpy(), r)
    assert np.array_equal(sizes.cpu().numpy(), c)
