"""Interleaving model of the cubic resolve pass with its per-tile table of
minima (Sec. II.C on the simple cubic lattice).

The merge's final trees are given.  A workgroup per tile takes its ids: an id
walks to its root (plain loads, which may return any value the entry held in the
launch), stores the root, and gives its key to its root's slot of the tile's
table: the slot's owner is set by a compare-and-swap from "free"; if the slot is
the root's, the key goes into the slot's minimum by an atomic, else (another
root's slot) straight to memory.  After the workgroup's barrier every owned
slot's minimum goes to memory.  A key goes to memory by an atomic minimum, if
memory's key as read past the caches is larger.

Every schedule must leave every id pointing at its root and each root's key equal
to its component's smallest.  A table read out without the barrier, a key whose
slot is another root's dropped, and a minimum stored plainly must be caught.
"""
import random

import pytest

from tests.test_cubic_merge_model import _case, _check, _merge

FREE, LARGEST = -1, 1 << 40


def _resolve(parent, key, tile_of, n_slots, rng, mistake=None):
    n, n_tiles = len(parent), max(tile_of) + 1
    G = [[p] for p in parent]  # values each parent entry held in this launch
    K = list(key)
    owner = [[FREE] * n_slots for _ in range(n_tiles)]
    least = [[LARGEST] * n_slots for _ in range(n_tiles)]
    waiting = [sum(t == j for t in tile_of) for j in range(n_tiles)]  # ids before the barrier

    def load(x):
        h = G[x]
        return h[rng.randrange(len(h))] if len(h) > 1 and rng.random() < 0.5 else h[-1]

    def take(root, k):
        now = K[root]
        yield
        if k < now:
            K[root] = min(K[root], k)
            yield

    def of_id(i):
        t = tile_of[i]
        x = i
        p = load(x)
        yield
        while p != x:
            x = p
            p = load(x)
            yield
        if x != i:
            G[i].append(x)
            yield
            h = x % n_slots
            was = owner[t][h]
            if was == FREE:
                owner[t][h] = x
            yield
            if was in (FREE, x):
                old = least[t][h]
                if mistake == "plain_minimum":
                    yield
                least[t][h] = min(old, key[i])
                yield
            elif mistake != "collision_dropped":
                yield from take(x, key[i])
        waiting[t] -= 1

    def of_slot(t, h):
        while waiting[t] and mistake != "no_barrier":
            yield
        if owner[t][h] != FREE:
            yield from take(owner[t][h], least[t][h])

    live = [of_id(i) for i in range(n)] + [of_slot(t, h) for t in range(n_tiles) for h in range(n_slots)]
    while live:
        k = rng.randrange(len(live))
        try:
            next(live[k])
        except StopIteration:
            live[k] = live[-1]
            live.pop()
    return [h[-1] for h in G], K


def _one(rng, n, mistake=None):
    key, pairs = _case(rng, n, n + n // 3)
    par = _merge(n, pairs, rng, False)
    tile_of = sorted(rng.randrange(3) for _ in range(n))
    par, K = _resolve(par, key, tile_of, rng.choice((1, 2, 8)), rng, mistake)
    _check(n, pairs, key, par, K)


@pytest.mark.parametrize("n", [6, 20, 60])
def test_resolve_with_a_table(n):
    rng = random.Random(n)
    for _ in range(200 if n < 60 else 50):
        _one(rng, n)


@pytest.mark.parametrize("mistake", ["no_barrier", "collision_dropped", "plain_minimum"])
def test_planted_mistakes_are_caught(mistake):
    rng = random.Random(23)
    for _ in range(3000):
        try:
            _one(rng, 24, mistake)
        except AssertionError:
            return
    pytest.fail(f"the planted mistake {mistake!r} was not exposed")
