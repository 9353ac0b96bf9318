"""The per-sweep records of tiled lattices against plain numpy counts of the
spins they describe (whole numbers: equal).

Rows shorter than one 16-site segment, of exactly one, one site past one, a
ragged last segment that overlaps the one before, a row end on a segment end,
states at and above 8 (not counted), one and several segments a thread, one
and several workgroups.
"""
import numpy as np
import pytest

import paper_1105_5804_amd as sw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _counts(s, ising):
    st = (s == 1).astype(np.uint8) if ising else s
    return [int((st == k).sum()) for k in range(8)]


def _nsat(s, axes):
    return sum(int((s == np.roll(s, -1, axis=a)).sum()) for a in axes)


@pytest.mark.parametrize("W,H,q,ising", [
    (2, 300, 2, True), (15, 90, 3, False), (16, 65, 2, False), (17, 129, 2, True), (31, 70, 8, False),
    (32, 200, 11, False), (130, 33, 4, False), (257, 95, 2, True), (1000, 70, 5, False), (2049, 2500, 3, False),
])
def test_square_records(W, H, q, ising):
    lat = sw.SWLattice(W, H, q=q, K=0.9, seed=77, ising=ising)
    for _ in range(3):
        rec = lat.sweep_history(1).cpu().numpy()[0]
        s = lat.spins.cpu().numpy()
        assert rec[2] == -1
        assert rec[3] == _nsat(s, (0, 1))
        assert rec[4:].tolist() == _counts(s, ising)
        o = lat.observables()
        assert (o["n_active_bonds"], o["n_clusters"], o["n_sat"]) == (rec[0], rec[1], rec[3])


@pytest.mark.parametrize("L,q,ising", [
    ((1, 1, 6), 2, True), ((7, 1, 5), 3, False), ((16, 3, 1), 2, True), ((20, 18, 2), 9, False), ((33, 70, 20), 3, False),
    ((160, 64, 48), 2, True), ((1030, 33, 130), 2, False),
])
def test_cubic_records(L, q, ising):
    lat = sw.CubicLattice(*L, q=q, K=0.5, seed=78, ising=ising)
    for _ in range(2):
        rec = lat.sweep(2, records=True).cpu().numpy()[1]
        s = lat.spins.cpu().numpy()
        assert rec[2] == _nsat(s, (0, 1, 2))
        assert rec[3:].tolist() == _counts(s, ising)
