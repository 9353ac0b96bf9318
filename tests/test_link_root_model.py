"""Interleaving model of the tile kernels' labels linked by one compare-and-swap
beside the union steps of other waves (Sec. II.B.2).

Waves own consecutive ranges of sites.  Each has labeled its own range (a site's
entry is its label, a site of the range at or below it) and kept the labels in
registers.  Then, with no barrier between the waves, a wave

  1. takes its bonds to the next range: it reads the far site's entry; if that
     is a label of the far range (at or past the range's first site), it swaps
     the label's entry from itself to the near site's label (one
     compare-and-swap).  The bond is met if the swap succeeded or found the near
     label already there; otherwise it is listed;
  2. unites its listed bonds (these, and bonds inside its range whose label
     offers lost) by union steps: two levels climbed, the larger of two roots
     put below the smaller by an atomic minimum, a lane with nothing to link
     halving its path.

In the small-lattice kernel (`pairs`) a bond joins any two sites: both entries
are read, and the larger label is swapped to the smaller.

A seeded random scheduler interleaves every load and atomic of all lanes.  Each
schedule must keep every parent at or below its child and end with the exact
partition, each root its component's smallest site.  A swap made of a load and
a store, a failed swap taken for met, a label outside the far range linked all
the same, and (pairs) the smaller label linked below the larger must be caught.
"""
import random

import pytest

from tests.test_union_model import _check, _components


def _case(rng, n, n_waves, pairs):
    """Entries (labels) of every site, bonds to link and bonds to unite."""
    per = n // n_waves
    P, first = [], []
    for x in range(n):
        w = min(x // per, n_waves - 1)
        first.append(w * per)
        own = [y for y in range(w * per, x) if P[y] == y]
        P.append(x if not own or rng.random() < 0.5 else rng.choice(own))
    link, unite = [], []
    for _ in range(n):
        u = rng.randrange(n)
        if pairs:
            link.append((u, rng.randrange(n)))
        elif first[u] + per < n and first[u] // per < n_waves - 1:
            link.append((u, rng.randrange(first[u] + per, min(n, first[u] + 2 * per))))
    for _ in range(n // 4):
        u = rng.randrange(n)
        same = [y for y in range(n) if first[y] == first[u]]
        unite.append((u, rng.choice(same)))
    return P, first, link, unite


def _lane(P, first, bond, linked, pairs, mistake):
    """One bond's events, as a generator (each yield ends one memory event)."""
    u, v = bond
    if linked:
        if pairs:
            up = P[u]
            yield
            low = P[v]
            yield
            up, low = min(up, low), max(up, low)
            if mistake == "larger_parent":
                up, low = low, up
            try_it = up != low
            met = not try_it
        else:
            up = first["label"][u]  # held in a register since the wave labeled its range
            low = P[v]
            yield
            try_it = mistake == "any_label" or low >= first["of"][v]
            met = False
        if try_it:
            got = P[low]
            if mistake == "load_and_store":
                yield
            if got == low:
                P[low] = up
                assert up <= low, "parent above its child"
            yield
            met = got == low or got == up or mistake == "failed_is_met"
        if met:
            return
    a = P[u]
    yield
    b = P[v]
    yield
    while True:
        pa = P[a]
        yield
        pb = P[b]
        yield
        ga = P[pa]
        yield
        gb = P[pb]
        yield
        roots = pa == a and pb == b
        move = roots and a != b
        hi, lo = max(a, b), min(a, b)
        at = hi if move else a
        old = P[at]
        P[at] = min(old, lo if move else ga)
        assert P[at] <= at, "parent above its child"
        yield
        if pa == pb or (roots and (not move or old == hi)):
            return
        a, b = (old, lo) if move else (ga, gb)


def _run(rng, n, n_waves, pairs, mistake=None):
    P, first, link, unite = _case(rng, n, n_waves, pairs)
    want = _components(P, link + unite)
    regs = {"label": list(P), "of": first}
    live = [_lane(P, regs, b, True, pairs, mistake) for b in link] + \
           [_lane(P, regs, b, False, pairs, mistake) for b in unite]
    events = 0
    while live:
        events += 1
        assert events < 100000, "no progress"
        k = rng.randrange(len(live))
        try:
            next(live[k])
        except StopIteration:
            live[k] = live[-1]
            live.pop()
    _check(P, want)


@pytest.mark.parametrize("pairs", [False, True], ids=["next_range", "pairs"])
@pytest.mark.parametrize("n,n_waves", [(8, 2), (24, 4), (64, 8)])
def test_links_beside_unions(n, n_waves, pairs):
    rng = random.Random(100 * n + n_waves + pairs)
    for _ in range(300 if n < 64 else 80):
        _run(rng, n, n_waves, pairs)


@pytest.mark.parametrize("mistake,pairs", [("load_and_store", False), ("failed_is_met", False), ("any_label", False),
                                           ("load_and_store", True), ("failed_is_met", True), ("larger_parent", True)])
def test_planted_mistakes_are_caught(mistake, pairs):
    rng = random.Random(17)
    for _ in range(3000):
        try:
            _run(rng, 24, 4, pairs, mistake)
        except AssertionError:
            return
    pytest.fail(f"{mistake}: no interleaving in 3000 trials exposed it")
