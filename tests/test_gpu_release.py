"""Blocks released while copies of their results are still queued: the copies
are held back by a bounded delay on the callers' streams, the arena has room
for no more than the blocks released, and the requests that take them over hold
something else."""
import numpy as np
import pytest

import paper_1105_5804_amd as sw

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIDE = 200
DELAY = 100_000_000  # clock ticks


def _served(srv, n):
    slots = {}
    while len(slots) < n:
        srv.pump()
        for slot, tag in srv.poll():
            slots[tag] = slot
    return slots


@pytest.mark.parametrize("batch_px", [0, 1 << 20], ids=["unbatched", "batched"])
def test_blocks_wait_for_every_streams_copies(batch_px):
    g = np.random.default_rng(31)
    images = [torch.from_numpy((g.random((SIDE, SIDE)) < p).astype(np.uint8)).pin_memory()
              for p in (0.5, 0.6, 0.3, 0.8)]
    want = [sw.ccl_label(img.cuda(), "sites_open") for img in images]
    probe = sw.CCLServer(64 << 20, sizes=True, max_inflight=2, n_streams=2, batch_px=batch_px)
    fp = probe.footprint(SIDE, SIDE)
    probe.close()
    tables = 0  # the arena's front holds the batch tables: the least that serves two requests
    while True:
        try:
            srv = sw.CCLServer(tables + 2 * fp, sizes=True, max_inflight=2, n_streams=2, batch_px=batch_px)
            srv.submit(0, images[0])
            srv.submit(1, images[1])
            if len(srv._inflight) == 2:
                break
            srv.close()
        except sw.SwccLError:
            pass
        tables += fp
    slots = _served(srv, 2)
    own = [torch.cuda.Stream(), torch.cuda.Stream()]
    copies = []
    for k, s in enumerate(own):
        with torch.cuda.stream(s):
            torch.cuda._sleep(DELAY)
            copies.append(srv.result(slots[k])[0].clone())
            srv.release(slots[k])
    srv.submit(2, images[2])
    srv.submit(3, images[3])
    slots = _served(srv, 2)
    for k in (2, 3):
        assert torch.equal(srv.result(slots[k])[0], want[k])
        srv.release(slots[k])
    torch.cuda.synchronize()
    for k in (0, 1):
        assert torch.equal(copies[k], want[k])
    srv.close()


def test_close_waits_for_the_copies():
    img = torch.from_numpy((np.random.default_rng(37).random((SIDE, SIDE)) < 0.6).astype(np.uint8)).pin_memory()
    want = sw.ccl_label(img.cuda(), "sites_open")
    srv = sw.CCLServer(16 << 20, sizes=True, max_inflight=1, n_streams=1)
    srv.submit(0, img)
    slot = _served(srv, 1)[0]
    own, done = torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(own):
        torch.cuda._sleep(DELAY)
        copy = srv.result(slot)[0].clone()
        done.record()
        srv.release(slot)
    srv.close()
    assert done.query()
    assert torch.equal(copy, want)
