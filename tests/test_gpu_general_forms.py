"""The kernels' general forms (any width) on lattices above the sizes up to which
a tile is worked by more waves, against the CPU oracle (whole numbers: equal):
odd and ragged widths of more than 256 square tiles, cubic extents that are odd
or twice an odd number with more than 512 and more than 1024 tiles, and served
batches of more than 256 tiles."""
import numpy as np
import pytest

import oracle
import paper_1105_5804_amd as sw
from paper_1105_5804_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _state(lat):
    s = lat.spins.cpu().numpy().reshape(-1)
    return (s == 1).astype(np.uint8) if lat.ising else s.astype(np.uint8)


def _equal(t, want):
    return np.array_equal(t.cpu().numpy().reshape(-1), want)


@pytest.mark.parametrize("W,H,q,K,few_b", [
    (2049, 1100, 3, 1.005, 0), (2050, 1100, 2, 0.8814, 0), (4097, 577, 2, 0.8814, 0), (2049, 1100, 2, 0.8814, 32),
    (2050, 1090, 2, 0.8814, 7),
])
@pytest.mark.parametrize("sizes", [False, True])
def test_square_sweeps(W, H, q, K, few_b, sizes):
    seed = wl.SEED_BASE | 0x4F1
    kw = dict(few_b=few_b, p_flip=0.6) if few_b else {}
    lat = sw.SWLattice(W, H, q=q, K=K, seed=seed, keep_labels=True, keep_bonds=True, sizes=sizes, **kw)
    T = oracle.threshold(K)
    st = oracle.init_states(W, H, q, seed)
    for t in range(3):
        rec = lat.sweep_history(1).cpu().numpy()[0]
        if few_b:
            st, bonds, labels, want, *_ = oracle.few_sweep(W, H, T, oracle.prob_threshold(0.6), few_b, seed, 0, t, st)
        else:
            st, bonds, labels, want = oracle.sw_sweep(W, H, q, T, seed, 0, t, st)
        assert _equal(lat.bonds, bonds) and _equal(lat.labels, labels), t
        assert np.array_equal(_state(lat), st), t
        nsat, counts = oracle.satisfied(W, H, q, st)
        assert rec[[0, 1, 3]].tolist() == [want[oracle.REC_ACTIVE], want[oracle.REC_NCLUST], nsat], t
        assert rec[4:4 + q].tolist() == [int(c) for c in counts[:q]], t
        if sizes:
            roots, n = np.unique(labels, return_counts=True)
            got_roots, got_sizes = lat.cluster_sizes()
            assert _equal(got_roots, roots) and _equal(got_sizes, n) and rec[2] == n.max(), t


@pytest.mark.parametrize("W,H", [(2049, 1100), (2050, 1090)])
@pytest.mark.parametrize("mode", ["sites_open", "bonds_open", "bonds_periodic"])
def test_labelings(W, H, mode):
    g = np.random.default_rng(W + H)
    if mode == "sites_open":
        inp = (g.random((H, W)) < 0.6).astype(np.uint8)
        want, n_want = oracle.label_sites(W, H, inp.reshape(-1))
    else:
        inp = g.integers(0, 4, (H, W), dtype=np.uint8)
        args = (oracle.OPEN,) if mode == "bonds_open" else ()
        want, n_want = oracle.label_bonds(W, H, inp.reshape(-1), *args)
    for sizes in (False, True):
        out = sw.ccl_label(torch.from_numpy(inp).cuda(), mode, sizes=sizes)
        assert _equal(out[0] if sizes else out, want)
        if sizes:
            r, c = np.unique(want[want >= 0], return_counts=True)
            assert out[3] == n_want == len(r) and _equal(out[1], r) and _equal(out[2], c)


# more than 512 tiles (770) and more than 1024 (1089)
CUBIC = [(321, 150, 100, 2), (322, 150, 100, 3), (323, 170, 130, 2), (322, 170, 130, 2)]


@pytest.mark.parametrize("Lx,Ly,Lz,q", CUBIC)
def test_cubic_sweeps(Lx, Ly, Lz, q):
    K, seed = (0.4433 if q == 2 else 0.55), wl.SEED_BASE | 0x4F2
    print(f"cubic {Lx} x {Ly} x {Lz}", flush=True)
    lat = sw.CubicLattice(Lx, Ly, Lz, q=q, K=K, seed=seed, ising=q == 2, keep_labels=True, keep_bonds=True)
    T = oracle.threshold(K)
    st = oracle.init_states3(Lx, Ly, Lz, q, seed)
    for t in range(2):
        rec = lat.sweep(1, records=True)
        st, bonds, labels, want = oracle.sw3_sweep(Lx, Ly, Lz, q, T, seed, 0, t, st)
        assert _equal(lat.bonds, bonds) and _equal(lat.labels, labels), t
        assert np.array_equal(_state(lat), st), t
        assert [int(v) for v in rec[0].cpu()] == [int(v) for v in want], t


@pytest.mark.parametrize("Lx,Ly,Lz,q", CUBIC)
def test_cubic_labelings(Lx, Ly, Lz, q):
    g = np.random.default_rng(Lx + Lz)
    for p in ((0.2488, 0.2488, 0.2488), (0.9, 0.1, 0.1), (0.1, 0.1, 0.9)):
        b = ((g.random((Lx * Ly * Lz, 3)) < np.array(p)) @ np.array([1, 2, 4])).astype(np.uint8)
        got, n = sw.ccl3_label(torch.from_numpy(b.reshape(Lz, Ly, Lx)).cuda())
        want, n_want = oracle.label_bonds3(Lx, Ly, Lz, b)
        assert n == n_want and _equal(got, want), p


@pytest.mark.parametrize("mode", ["sites_open", "bonds_open", "bonds_periodic"])
@pytest.mark.parametrize("sizes", [False, True])
def test_served_batch_of_many_tiles(mode, sizes):
    g = np.random.default_rng(29)
    n = 14  # of up to 32 tiles each, labeled together
    srv = sw.CCLServer(256 << 20, mode=mode, sizes=sizes, max_inflight=n, n_streams=2, batch_px=1 << 20)
    images = []
    for k in range(n):
        W, H = 480 + k, 440 + 3 * k
        images.append((g.random((H, W)) < 0.6).astype(np.uint8) if mode == "sites_open"
                      else g.integers(0, 4, (H, W), dtype=np.uint8))
        srv.submit(k, torch.from_numpy(images[-1]).pin_memory())
    got = {}
    while srv.pending:
        srv.pump()
        for slot, tag in srv.poll():
            lab, roots, szs, count = srv.result(slot)
            got[tag] = (lab.cpu(), roots.cpu() if sizes else None, szs.cpu() if sizes else None, count)
            srv.release(slot)
    srv.close()
    for k, img in enumerate(images):
        H, W = img.shape
        if mode == "sites_open":
            want, _ = oracle.label_sites(W, H, img.reshape(-1))
        else:
            want, _ = oracle.label_bonds(W, H, img.reshape(-1), *((oracle.OPEN,) if mode == "bonds_open" else ()))
        r, c = np.unique(want[want >= 0], return_counts=True)
        lab, roots, szs, count = got[k]
        assert count == len(r) and _equal(lab, want), k
        if sizes:
            assert _equal(roots, r) and _equal(szs, c), k
