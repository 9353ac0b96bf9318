"""The active bonds and clusters of a record, which the observables kernel adds
up from the tiles' counters, against the bond bytes and labels of the same sweep
(whole numbers: equal), on lattices of one and of several of its workgroups."""
import numpy as np
import pytest

import paper_1105_5804_amd as sw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _bits(bonds):
    return int(np.unpackbits(bonds.cpu().numpy().reshape(-1)).sum())


def _distinct(labels):
    return int(torch.unique(labels).numel())


@pytest.mark.parametrize("W,H,q,ising", [
    (2, 300, 2, True), (130, 33, 4, False), (257, 95, 2, True), (2049, 2500, 3, False), (6000, 3001, 2, True),
])
def test_square(W, H, q, ising):
    lat = sw.SWLattice(W, H, q=q, K=0.9, seed=79, ising=ising, keep_bonds=True, keep_labels=True)
    for _ in range(2):
        rec = lat.sweep_history(3).cpu().numpy()[2]
        assert rec[0] == _bits(lat.bonds) and rec[1] == _distinct(lat.labels)


@pytest.mark.parametrize("L,q,ising", [
    ((1, 1, 6), 2, True), ((33, 70, 20), 3, False), ((160, 64, 48), 2, True), ((1030, 33, 130), 2, False),
])
def test_cubic(L, q, ising):
    lat = sw.CubicLattice(*L, q=q, K=0.5, seed=80, ising=ising, keep_bonds=True, keep_labels=True)
    for _ in range(2):
        rec = lat.sweep(3, records=True).cpu().numpy()[2]
        assert rec[0] == _bits(lat.bonds) and rec[1] == _distinct(lat.labels)
