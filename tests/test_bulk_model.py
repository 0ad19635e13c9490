"""CPU model of a bulk insert's commit beside plain inserts, and the arithmetic of its split.

The model: one base slab of unique-key pairs. Every slot read, swap and store is a step of a random
schedule of several inserters, so a slab is never read at one instant.
  plain inserter  reads the slots in any order; its key's slot: swap in the new value; else swap
                  into the first slot that read empty or locked; a swap that meets the lock reads
                  the slab again; one that meets another key walks on.
  bulk inserter   reads the slots; swaps the first empty one to the lock (if that fails it leaves
                  its keys to plain inserts), stores the later slots' pairs in any order, then the
                  locked slot's pair.
Whatever the schedule, no key is in two slots, empty slots are a suffix, and no lock remains."""
import random

import pytest

EMPTY, LOCK, M = "empty", "lock", 6


class Slab:
    def __init__(self, held):
        self.s = list(held) + [EMPTY] * (M - len(held))

    def cas(self, i, expect, new):
        old = self.s[i]
        if old == expect:
            self.s[i] = new
        return old


def plain(slab, key, val, log, obey=True):
    while True:
        seen = [None] * M
        order = list(range(M))
        random.shuffle(order)
        for i in order:
            seen[i] = slab.s[i]
            yield
        at = next((i for i, p in enumerate(seen) if p[0] == key), None)
        if at is not None:
            if slab.cas(at, seen[at], (key, val)) == seen[at]:
                log.append(key)
                return
            yield
            continue
        i = next((i for i, p in enumerate(seen) if p == EMPTY or (obey and p == LOCK)), None)
        if i is None:
            return  # the list's next slab: not modelled
        again = False
        while i < M and not again:
            yield
            old = slab.cas(i, EMPTY, (key, val))
            if old == EMPTY:
                log.append(key)
                return
            if old == LOCK and obey:
                again = True
            elif old[0] == key:
                yield
                if slab.cas(i, old, (key, val)) == old:
                    log.append(key)
                    return
                again = True
            else:
                i += 1
        if not again:
            return


def bulk(slab, pairs, log, obey=True):
    seen = [None] * M
    for i in random.sample(range(M), M):
        seen[i] = slab.s[i]
        yield
    held = {p[0] for p in seen if p not in (EMPTY, LOCK)}
    first = next((i for i, p in enumerate(seen) if p == EMPTY), M)
    new = [p for p in pairs if p[0] not in held]
    left = [p for p in pairs if p[0] in held]
    if LOCK in seen:
        new, left = [], pairs
    fits = new[: M - first]
    left = left + new[len(fits):]
    if fits:
        yield
        if slab.cas(first, EMPTY, LOCK if len(fits) > 1 else fits[0]) == EMPTY:
            for j in random.sample(range(1, len(fits)), len(fits) - 1):
                yield
                slab.s[first + j] = fits[j]
            yield
            slab.s[first] = fits[0]
            log.extend(p[0] for p in fits)
        else:
            left = left + fits
    for k, v in left:
        yield from plain(slab, k, v, log, obey)


def run(seed, obey=True):
    """Whether the end state is sound after one random schedule."""
    random.seed(seed)
    slab = Slab([(k, 0) for k in range(random.randrange(3))])
    log = []
    keys = list(range(5))
    todo = [bulk(slab, [(k, 10 + k) for k in random.sample(keys, 3)], log, obey)
            for _ in range(random.choice([1, 2]))]
    todo += [plain(slab, random.choice(keys), 20 + i, log, obey) for i in range(3)]
    steps = 0
    while todo:
        g = random.choice(todo)
        steps += 1
        assert steps < 100000, "a wait that does not end"
        try:
            next(g)
        except StopIteration:
            todo.remove(g)
    held = [p[0] for p in slab.s if p != EMPTY]
    n = len(held)
    return (LOCK not in slab.s and all(p != EMPTY for p in slab.s[:n])
            and len(set(held)) == n and set(log) <= set(held))


def test_commit_beside_plain_inserts():
    assert all(run(s) for s in range(6000))


def test_inserters_that_ignore_the_lock_are_caught():
    assert not all(run(s, obey=False) for s in range(6000))


@pytest.mark.parametrize("d", [1, 2, 3, 107, 4096, 54343, 217316, 3477982, 2**31, 2**32 - 1])
def test_quotient_by_multiplication(d):
    """x // d for 32-bit x from the high half of x * floor(2^32 / d) and one correction."""
    m = 0xFFFFFFFF if d <= 1 else (1 << 32) // d
    rng = random.Random(d)
    xs = [0, 1, d - 1, d, d + 1, 2**32 - 1, 2**32 - 2] + [rng.randrange(2**32) for _ in range(20000)]
    xs += [min(2**32 - 1, d * rng.randrange(2**32 // d + 1) + e) for e in (0, 1) for _ in range(5000)]
    xs += [max(0, d * rng.randrange(2**32 // d + 1) - 1) for _ in range(5000)]
    for x in xs:
        if x >= 2**32:
            continue
        q = (x * m) >> 32
        r = x - q * d
        assert 0 <= r < 2 * d
        if r >= d:
            q, r = q + 1, r - d
        assert (q, r) == divmod(x, d)


@pytest.mark.parametrize("parts,tile", [(1, 4096), (2, 4096), (2043, 16384), (2048, 16384),
                                        (15872, 32768)])
def test_two_counts_per_word(parts, tile):
    """Part counts kept as 16-bit pairs become starts, the last word's end included."""
    row = parts // 2 + 1
    rng = random.Random(parts)
    p = [rng.randrange(parts) for _ in range(tile)]
    if parts == 2:
        p = [1] * tile  # one part holds the whole tile
    cnt = [0] * row
    for x in p:
        cnt[x >> 1] += 1 << (16 * (x & 1))
    assert all(c < 1 << 32 for c in cnt)
    at, starts = 0, []
    for c in cnt:
        starts += [at, at + (c & 0xFFFF)]
        at += (c & 0xFFFF) + (c >> 16)
    assert at == tile < 1 << 16 and len(starts) > parts and starts[parts] == tile
    for x in {0, parts // 2, parts - 1}:
        assert starts[x + 1] - starts[x] == p.count(x)
