"""The calls that users of this framework make, as measured cases.

Six kinds, each through the public entry points:

sweep   Swendsen-Wang sweeps of one periodic square lattice (``SWLattice``):
        a simulation calls ``sweep`` or ``sweep_history`` over and over on an
        equilibrated lattice, with the arrays it keeps (labels, bonds, cluster
        sizes) or with the few-cluster update.
batch   many independent lattices swept together (``SWBatch``).
cubic   sweeps of one periodic simple cubic lattice (``CubicLattice``).
ccl     labeling of one image or bond array on the device (``ccl_label``).
ccl3    labeling of given bonds of a cubic lattice (``ccl3_label``).
serve   a burst of host images through the labeling server (``CCLServer``),
        results copied out of the server's arena and released.

Every output is a whole number (spins, labels, bond bytes, counts), the same
for every correct implementation, so there is no 64-bit value to compare with.
"""
import math

import numpy as np
import torch

import paper_1105_5804_amd as sw
from paper_1105_5804_amd import workloads as wl

EQUILIBRATE = 20        # sweeps before the lattice is handed over, as a simulation's own warm-up
K3_ISING = 2.0 * sw.BETA_C_ISING_3D
BURST_MIN_SIDE = 64


def listed():
    return [
        # the smallest simulation: the paper's L = 64 Ising lattice, energy and
        # magnetisation recorded after every sweep
        dict(name="ising64_records", kind="sweep", W=64, H=64, q=2, beta=1.0, sweeps=100, records=True, labels=False,
             bonds=False, sizes=False, few_b=0),
        # a mid-size Potts lattice whose clusters are analysed (labels, roots
        # and sizes after the call): few tiles, so launches and latency count
        dict(name="potts512_sizes", kind="sweep", W=512, H=500, q=3, beta=1.0, sweeps=4, records=False, labels=True,
             bonds=False, sizes=True, few_b=0),
        # the few-cluster update on an odd width and height, with records, a
        # little above the critical temperature
        dict(name="few2049_records", kind="sweep", W=2049, H=1537, q=2, beta=0.95, sweeps=4, records=True,
             labels=False, bonds=False, sizes=False, few_b=32),
        # the measurement series at L = 4096 with the packed bonds kept
        dict(name="ising4096_records", kind="sweep", W=4096, H=4096, q=2, beta=1.0, sweeps=10, records=True,
             labels=False, bonds=True, sizes=False, few_b=0),
        # the benchmark lattice, one sweep a call
        dict(name="potts16384", kind="sweep", W=16384, H=16384, q=3, beta=1.0, sweeps=1, records=False, labels=False,
             bonds=False, sizes=False, few_b=0),
        # replicas and temperatures: 256 lattices of side 32 .. 1024 swept
        # together, replayed as graphs
        dict(name="batch256", kind="batch", n=256, sweeps=8, graph=True),
        # a small cubic Potts lattice with ragged tiles, in the ordered phase,
        # records after every sweep
        dict(name="cubic100_records", kind="cubic", Lx=100, Ly=75, Lz=61, q=3, K=0.6, sweeps=4, records=True,
             labels=False),
        # the critical Ising model on the large cubic lattice
        dict(name="cubic512", kind="cubic", Lx=512, Ly=512, Lz=512, q=2, K=K3_ISING, sweeps=1, records=False,
             labels=False),
        # one segmentation call on an image of odd width, with component sizes
        dict(name="image1001_sizes", kind="ccl", W=1001, H=1333, mode="sites_open", p=0.55, sizes=True),
        # the large labeling pass: bond percolation at its threshold
        dict(name="percolation16384", kind="ccl", W=16384, H=16384, mode="bonds_periodic", p=0.5, sizes=False),
        # bond percolation on the cubic lattice at its threshold
        dict(name="cubic_percolation256", kind="ccl3", Lx=256, Ly=256, Lz=256, p=0.2488),
        # a burst of requests of mixed sizes, batched by the server
        dict(name="serve24", kind="serve", n=24, max_side=1024, p=0.58, batch_px=1 << 20),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["sweep", "sweep", "sweep", "batch", "cubic", "cubic", "ccl", "ccl", "ccl3", "serve"])
    if kind == "sweep":
        W, H = _log_int(rng, 24, 8192), _log_int(rng, 24, 8192)
        W = W + W % 2 if rng.random() < 0.5 else W
        sweeps = rng.choice([1, 2, 4]) if W * H <= 1 << 24 else 1
        few = rng.random() < 0.2
        option = rng.choice(["none", "none", "labels", "bonds", "sizes"])
        return dict(kind=kind, W=W, H=H, q=2 if few else rng.choice([2, 2, 3, 4, 10]), beta=rng.uniform(0.6, 1.4),
                    sweeps=sweeps, records=rng.random() < 0.4, labels=option == "labels",
                    bonds=option == "bonds", sizes=option == "sizes", few_b=_log_int(rng, 4, 256) if few else 0)
    if kind == "batch":
        return dict(kind=kind, n=_log_int(rng, 4, 256), sweeps=rng.choice([1, 3, 8]), graph=rng.random() < 0.5)
    if kind == "cubic":
        side = [_log_int(rng, 12, 384) for _ in range(3)]
        return dict(kind=kind, Lx=side[0], Ly=side[1], Lz=side[2], q=rng.choice([2, 2, 3]), K=rng.uniform(0.3, 0.65),
                    sweeps=rng.choice([1, 2, 4]) if side[0] * side[1] * side[2] <= 1 << 23 else 1,
                    records=rng.random() < 0.5, labels=rng.random() < 0.3)
    if kind == "ccl":
        return dict(kind=kind, W=_log_int(rng, 24, 8192), H=_log_int(rng, 24, 8192),
                    mode=rng.choice(["sites_open", "sites_open", "bonds_open", "bonds_periodic"]),
                    p=rng.uniform(0.3, 0.75), sizes=rng.random() < 0.5)
    if kind == "ccl3":
        side = [_log_int(rng, 12, 384) for _ in range(3)]
        return dict(kind=kind, Lx=side[0], Ly=side[1], Lz=side[2], p=rng.uniform(0.1, 0.5))
    return dict(kind=kind, n=_log_int(rng, 4, 24), max_side=_log_int(rng, 128, 1024), p=rng.uniform(0.4, 0.7),
                batch_px=rng.choice([0, 1 << 20]))


def _sides(case):
    """Sides of a batch's lattices: 32 .. 1024 in turn."""
    return [32 << (j % 6) for j in range(case["n"])]


def _burst(case):
    """(W, H) of a burst's images: log-uniform sides, the same for every seed."""
    g = np.random.default_rng(case["n"] * 1000003 + case["max_side"])
    u = g.random((case["n"], 2))
    side = np.exp(math.log(BURST_MIN_SIDE) + math.log(case["max_side"] / BURST_MIN_SIDE) * u)
    return [(int(round(w)), int(round(h))) for w, h in side]


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _occupied(shape, p, g):
    return (torch.rand(shape, generator=g, device="cuda") < p).to(torch.uint8)


def _padded(values, length):
    """A list of clusters as an array of fixed length, -1 past its end, as a program stores it beside others."""
    return torch.nn.functional.pad(values, (0, length - values.numel()), value=-1)


def prepare(case, seed):
    key = wl.SEED_BASE + 0x10000 + seed
    kind = case["kind"]
    if kind == "sweep":
        K = case["beta"] * math.log1p(math.sqrt(case["q"]))
        lat = sw.SWLattice(case["W"], case["H"], q=case["q"], K=K, seed=key, keep_labels=case["labels"] or case["sizes"],
                           keep_bonds=case["bonds"], sizes=case["sizes"], few_b=case["few_b"],
                           p_flip=0.5 if case["few_b"] else 0.0)
        lat.sweep(EQUILIBRATE)
        return dict(case, lattice=lat)
    if kind == "batch":
        beta = wl.rng(key).uniform(0.9, 1.1, size=case["n"])
        specs = [dict(W=L, H=L, q=2, ising=True, K=wl.K_ISING_C * float(b), seed=key + j, stream_id=j)
                 for j, (L, b) in enumerate(zip(_sides(case), beta))]
        batch = sw.SWBatch(specs)
        batch.sweep(EQUILIBRATE)
        return dict(case, batch=batch)
    if kind == "cubic":
        lat = sw.CubicLattice(case["Lx"], case["Ly"], case["Lz"], q=case["q"], K=case["K"], seed=key,
                              keep_labels=case["labels"])
        lat.sweep(EQUILIBRATE)
        return dict(case, lattice=lat)
    g = _generator(seed)
    if kind == "ccl":
        shape = (case["H"], case["W"])
        if case["mode"] == "sites_open":
            inp = _occupied(shape, case["p"], g)
        else:
            inp = _occupied(shape, case["p"], g) | (_occupied(shape, case["p"], g) << 1)
        return dict(case, input=inp)
    if kind == "ccl3":
        shape = (case["Lz"], case["Ly"], case["Lx"])
        bonds = _occupied(shape, case["p"], g)
        for axis in (1, 2):
            bonds |= _occupied(shape, case["p"], g) << axis
        return dict(case, input=bonds)
    r = wl.rng(key)
    images = []
    for W, H in _burst(case):
        img = torch.empty((H, W), dtype=torch.uint8, pin_memory=True)
        img.copy_(torch.from_numpy((r.random((H, W)) < case["p"]).astype(np.uint8)))
        images.append(img)
    server = sw.CCLServer(1 << 30, mode="sites_open", sizes=True, max_inflight=64, n_streams=4,
                          batch_px=case["batch_px"])
    return dict(case, images=images, server=server)


def _run_serve(state):
    server, images = state["server"], state["images"]
    for tag, img in enumerate(images):
        server.submit(tag, img)
    start = np.cumsum([0] + [img.numel() for img in images])
    labels, roots, sizes = (torch.full((int(start[-1]),), -1, dtype=torch.int32, device="cuda") for _ in range(3))
    counts = np.zeros(len(images), dtype=np.int64)
    done = 0
    while done < len(images):
        server.pump()
        for slot, tag in server.poll():
            lab, rts, szs, n = server.result(slot)
            at = int(start[tag])
            labels[at:int(start[tag + 1])] = lab.reshape(-1)
            roots[at:at + n] = rts
            sizes[at:at + n] = szs
            counts[tag] = n
            server.release(slot)
            done += 1
    return {"labels": labels, "roots": roots, "sizes": sizes, "counts": counts}


def run(state):
    kind = state["kind"]
    if kind in ("sweep", "cubic"):
        lat = state["lattice"]
        records = None
        if kind == "cubic":
            records = lat.sweep(state["sweeps"], records=state["records"])
        elif state["records"]:
            records = lat.sweep_history(state["sweeps"])
        else:
            lat.sweep(state["sweeps"])
        out = {"spins": lat.spins}
        if records is not None:
            out["records"] = records
        if lat.labels is not None:
            out["labels"] = lat.labels
        if lat.bonds is not None:
            out["bonds"] = lat.bonds
        if state.get("sizes"):
            roots, sizes = lat.cluster_sizes()
            out["roots"], out["sizes"] = _padded(roots, lat.roots.numel()), _padded(sizes, lat.sizes.numel())
        return out
    if kind == "batch":
        batch = state["batch"]
        batch.sweep(state["sweeps"], graph=state["graph"])
        return torch.cat([s.reshape(-1) for s in batch.spins])
    if kind == "ccl":
        if not state["sizes"]:
            return sw.ccl_label(state["input"], state["mode"])
        labels, roots, sizes, n = sw.ccl_label(state["input"], state["mode"], sizes=True)
        return {"labels": labels, "roots": _padded(roots, labels.numel()), "sizes": _padded(sizes, labels.numel()), "n": n}
    if kind == "ccl3":
        labels, n = sw.ccl3_label(state["input"])
        return {"labels": labels, "n": n}
    return _run_serve(state)


# Integer operations of a site's bond draws: a Philox4x32-10 block (ten rounds
# of two wide products and four exclusive-ors) gives four words; the square
# lattice takes two a site, the cubic lattice three.
OPS_2D, OPS_3D = 40, 60


def work(case):
    kind = case["kind"]
    if kind == "sweep":
        N, n = case["W"] * case["H"], case["sweeps"]
        on_chip = N <= 128 * 64 and not case["sizes"] and not case["few_b"]  # stays there between a call's sweeps
        moved = 2 * N * (1 if on_chip else n)
        moved += 4 * N * (case["labels"] or case["sizes"]) + N * case["bonds"]
        return {"bytes": moved, "flops": OPS_2D * N * n}
    if kind == "batch":
        N, n = sum(L * L for L in _sides(case)), case["sweeps"]
        return {"bytes": 2 * N * n, "flops": OPS_2D * N * n}
    if kind == "cubic":
        N, n = case["Lx"] * case["Ly"] * case["Lz"], case["sweeps"]
        return {"bytes": 2 * N * n + 4 * N * case["labels"], "flops": OPS_3D * N * n}
    if kind == "ccl":
        return {"bytes": 5 * case["W"] * case["H"], "flops": 0}
    if kind == "ccl3":
        return {"bytes": 5 * case["Lx"] * case["Ly"] * case["Lz"], "flops": 0}
    return {"bytes": 5 * sum(W * H for W, H in _burst(case)), "flops": 0}
