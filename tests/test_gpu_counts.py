"""Counts handed to the host: the cluster count of a lattice with sizes and of
served requests, batched and not, against the labels they belong to, with slots
and arena blocks reused while copies of the results before are still queued."""
import ctypes

import numpy as np
import pytest

import paper_1105_5804_amd as sw
from paper_1105_5804_amd import _lib

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("W,H,few_b", [(40, 30, 0), (300, 131, 0), (4096, 1100, 0), (130, 70, 16)])
def test_cluster_count(W, H, few_b):
    kw = dict(few_b=few_b, p_flip=0.5) if few_b else {}
    lat = sw.SWLattice(W, H, q=2, seed=5, keep_labels=True, sizes=True, **kw)
    n = ctypes.c_int64()
    assert _lib.lib().sw_cluster_count(lat._h, ctypes.byref(n), None) == _lib.SW_OK and n.value == -1
    for _ in range(2):
        lat.sweep(2)
        roots, sizes = lat.cluster_sizes()
        r, c = np.unique(lat.labels.cpu().numpy(), return_counts=True)
        assert np.array_equal(roots.cpu().numpy(), r) and np.array_equal(sizes.cpu().numpy(), c)
        assert lat.observables()["n_clusters"] == len(r)
    plain = sw.SWLattice(W, H, q=2, seed=5)
    assert _lib.lib().sw_cluster_count(plain._h, ctypes.byref(n), None) == _lib.SW_ERR_ARG


@pytest.mark.parametrize("batch_px,sizes", [(0, True), (1 << 14, True), (1 << 14, False)])
def test_served_counts(batch_px, sizes):
    g = np.random.default_rng(3)
    srv = sw.CCLServer(8 << 20, mode="sites_open", sizes=sizes, max_inflight=6, n_streams=3, batch_px=batch_px)
    images = [(g.random((int(h), int(w))) < 0.6).astype(np.uint8) for w, h in g.integers(20, 260, (40, 2))]
    for k, img in enumerate(images):
        srv.submit(k, torch.from_numpy(img))
    kept = {}
    while srv.pending:
        srv.pump()
        for slot, tag in srv.poll():
            lab, roots, szs, n = srv.result(slot)
            kept[tag] = (lab.clone(), n, roots.clone() if sizes else None)
            srv.release(slot)
    for k, img in enumerate(images):
        lab, n, roots = kept[k]
        want = sw.ccl_label(torch.from_numpy(img).cuda(), "sites_open")
        assert torch.equal(lab, want)
        u = torch.unique(want[want >= 0])
        assert n == u.numel()
        if sizes:
            assert torch.equal(roots.long(), u.long())
    srv.close()
