"""Timed workloads of the slab hash, each a pass through the Python entry points as a program
that uses the table calls them.

A case is a dict of plain values whose "kind" says what the pass does:

lookup    one search of a batch of keys in a resident table
build     a table emptied and bulk-built, then the first lookups in it
grow      a table emptied and filled by a stream of insert batches (incremental insertion), then
          a first batch of lookups
phased    a table emptied, built, searched, a quarter of its keys deleted, searched again
mixed     concurrent batches of inserts, deletes and searches on a resident table, then a flush
batched   one launch of per-table mixed batches over many tables
multiset  a table with duplicate keys: copies inserted, SEARCHALL, DELETEALL, search

Every pass leaves its state as a later pass needs it: phases that fill a table empty it first,
the mixed batches delete what they inserted and put back what they deleted, and a repeated
batched launch replaces the pairs that it inserted the first time.

Keys are a seeded bijection of counters, so key sets from disjoint counter ranges are disjoint
(the paper's workloads are uniform random keys); values are a mix of the key. Skewed queries are
Zipf(1.1) ranks over the table's keys, the distribution of the served workload.
"""
import functools
import math
import random

import torch

from paper_1710_11246_amd import autotune as A
from paper_1710_11246_amd import slabhash as S

DEV = "cuda"
M32 = 0xFFFFFFFF
PAIRS = {False: 31, True: 62}  # entries of a slab: key/value pairs, or keys alone
SEARCH, INSERT, DELETE = S.SH_OP_SEARCH, S.SH_OP_INSERT, S.SH_OP_DELETE


def listed():
    return [
        # a request handler looking up a handful of popular keys: latency of one small call
        dict(name="lookup_1k", kind="lookup", keys=1 << 20, util=0.6, queries=1000, hit=0.9,
             skew=True),
        # the paper's bulk search at its size: every key present
        dict(name="lookup_4m", kind="lookup", keys=1 << 22, util=0.6, queries=1 << 22, hit=1.0,
             skew=False),
        # mostly absent keys, in a table packed to 0.8: lists of about three slabs
        dict(name="lookup_4m_long_lists", kind="lookup", keys=1 << 22, util=0.8,
             queries=1 << 22, hit=0.1, skew=False),
        # a join side: half the probes present, in a table far larger than the caches
        dict(name="lookup_64m", kind="lookup", keys=1 << 26, util=0.6, queries=1 << 26, hit=0.5,
             skew=False),
        # the small configuration of the benchmark: 2^16 keys in 2^12 buckets
        dict(name="phased_64k", kind="phased", keys=1 << 16, buckets=1 << 12, queries=1 << 16,
             keys_only=False),
        # a set of keys without values, odd sizes
        dict(name="phased_set_1m", kind="phased", keys=1000003, buckets=27001, queries=500009,
             keys_only=True),
        # the paper's bulk build at its size
        dict(name="build_4m", kind="build", keys=1 << 22, util=0.6, duplicate=0.0,
             queries=1 << 18),
        # an index built from scratch for a large resident table
        dict(name="build_64m", kind="build", keys=1 << 26, util=0.6, duplicate=0.0,
             queries=1 << 22),
        # incremental insertion: 16 batches of 2^16, final utilisation 0.65
        dict(name="grow_1m", kind="grow", keys=1 << 20, util=0.65, batches=16, queries=1 << 16),
        # the concurrent benchmark's distribution (20% inserts, 20% deletes, 60% searches)
        dict(name="mixed_64k", kind="mixed", keys=1 << 20, util=0.6, batches=4, ops=1 << 16,
             update=0.4),
        # the batched form: 256 tables, one batch each, one launch
        dict(name="batched_256", kind="batched", tables=256, keys=1 << 25, ops=5 << 19),
        # 2^18 keys with four copies each
        dict(name="multiset_256k", kind="multiset", keys=1 << 18, copies=4, util=0.6),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], log-uniform and mostly odd."""
    v = int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))
    return min(hi, max(lo, v | (rng.random() < 0.8)))


def draw(rng):
    kind = rng.choice(["lookup", "lookup", "lookup", "build", "build", "grow", "phased",
                       "mixed", "batched", "multiset"])
    util = rng.choice([0.2, 0.4, 0.5, 0.6, 0.6, 0.65, 0.8])
    if kind == "lookup":
        return dict(kind=kind, keys=_log(rng, 1 << 16, 1 << 25), util=util,
                    queries=_log(rng, 64, 1 << 25), hit=rng.choice([0.1, 0.5, 0.9, 1.0]),
                    skew=rng.random() < 0.3)
    if kind == "build":
        n = _log(rng, 1 << 14, 1 << 25)
        return dict(kind=kind, keys=n, util=util, duplicate=rng.choice([0.0, 0.0, 0.25]),
                    queries=max(64, n // 16))
    if kind == "grow":
        return dict(kind=kind, keys=_log(rng, 1 << 16, 1 << 22), util=util,
                    batches=rng.choice([8, 16, 32]), queries=_log(rng, 1 << 10, 1 << 17))
    if kind == "phased":
        n, ko = _log(rng, 1 << 12, 1 << 21), rng.random() < 0.5
        return dict(kind=kind, keys=n, buckets=max(1, n // _log(rng, 6, 40)),
                    queries=_log(rng, 1 << 12, 1 << 21), keys_only=ko)
    if kind == "mixed":
        return dict(kind=kind, keys=_log(rng, 1 << 18, 1 << 23), util=util, batches=4,
                    ops=_log(rng, 1 << 10, 1 << 17), update=rng.choice([0.2, 0.4, 1.0]))
    if kind == "batched":
        t = _log(rng, 8, 512)
        return dict(kind=kind, tables=t, keys=t * _log(rng, 1 << 12, 1 << 16),
                    ops=t * _log(rng, 1 << 8, 1 << 13))
    return dict(kind=kind, keys=_log(rng, 1 << 12, 1 << 20), copies=rng.choice([2, 4]),
                util=rng.choice([0.4, 0.6]))


# --------------------------------------------------------------------------------------------
# Inputs

def _mix(x):
    """A bijection of the 32-bit integers (MurmurHash3's finaliser), on int64 tensors."""
    x = x ^ (x >> 16)
    x = (x * 0x85EBCA6B) & M32
    x = x ^ (x >> 13)
    x = (x * 0xC2B2AE35) & M32
    return x ^ (x >> 16)


def _i32(x):
    return torch.where(x >= 1 << 31, x - (1 << 32), x).to(torch.int32)


def _keys(seed, start, n):
    """Keys of the counters start .. start + n - 1 (below 2^32 - 2): distinct, and none of the
    two values that tables reserve, whose places the keys of the last two counters take."""
    s1 = (seed * 0x9E3779B1 + 0x7F4A7C15) & M32
    s2 = (seed * 0x85EBCA77 + 0x165667B1) & M32

    def image(x):
        return _mix(_mix(x ^ s1) ^ s2)

    k = image(torch.arange(start, start + n, dtype=torch.int64, device=DEV))
    s1, s2 = image(torch.tensor([M32, M32 - 1], dtype=torch.int64, device=DEV)).unbind()
    k, at = (torch.where(k == M32, torch.where(s1 == M32 - 1, s2, s1), k), k)
    return _i32(torch.where(at == M32 - 1, torch.where(s2 == M32, s1, s2), k))


def _vals(keys, salt=0):
    return _i32(_mix((keys.to(torch.int64) & M32) ^ (0x51ED270B + salt)))


def _gen(seed, what):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + what)


def _hash(seed):
    r = random.Random(seed * 7919 + 13)
    return r.randrange(1, S.SH_HASH_PRIME), r.randrange(S.SH_HASH_PRIME)


@functools.lru_cache(maxsize=None)
def _geometry(n, util, extra=0):
    """Buckets for n keys at a memory utilisation, and pool slabs with room for `extra` more."""
    b = A.buckets_for_utilisation(n, util)
    return b, A.pool_slabs_for(n + extra, b)


def _ranks(n, count, gen, skew):
    """`count` key indices below n: uniform, or Zipf(1.1) by the power law's inverse."""
    u = torch.rand(count, dtype=torch.float64, device=DEV, generator=gen)
    if not skew:
        return (u * n).to(torch.int64).clamp_(max=n - 1)
    top = float(n) ** -0.1
    return ((1.0 + u * (top - 1.0)) ** -10.0).to(torch.int64).sub_(1).clamp_(0, n - 1)


def _queries(case, seed, keys, lo=0):
    """(queries, present): `hit` of them keys of the table from index lo up, the rest absent,
    in random order; an all-hit uniform batch as long as the table asks for each key once."""
    n, q, hit = keys.numel(), case["queries"], case.get("hit", 0.5)
    g = _gen(seed, 1)
    if hit == 1.0 and q == n and not case.get("skew"):
        at = torch.randperm(n, device=DEV, generator=g)
        return keys[at], torch.ones(n, dtype=torch.bool, device=DEV)
    out = _keys(seed, n + (1 << 26), q)
    present = torch.rand(q, device=DEV, generator=g) < hit
    at = lo + _ranks(n - lo, q, g, case.get("skew"))
    return torch.where(present, keys[at], out), present


def _found(queries, present, keys_only=False):
    v = torch.where(present, queries if keys_only else _vals(queries), -1)
    return v.to(torch.int64), present.to(torch.int64)


# --------------------------------------------------------------------------------------------
# One function per kind: (state, expected results). The state has the inputs and the table.

def _fill(t, keys, vals):
    for i in range(0, keys.numel(), 1 << 26):
        t.insert(keys[i:i + (1 << 26)], None if vals is None else vals[i:i + (1 << 26)],
                 status=False)


def _lookup(case, seed, table):
    keys = _keys(seed, 0, case["keys"])
    q, present = _queries(case, seed, keys)
    st = dict(q=q)
    if table:
        st["t"] = S.SlabHash(*_geometry(case["keys"], case["util"]), *_hash(seed))
        _fill(st["t"], keys, _vals(keys))
    return st, lambda: _found(q, present)


def _build(case, seed, table):
    n = case["keys"]
    keys = _keys(seed, 0, n)
    m = int(n * case["duplicate"])
    if m:  # the last pairs repeat keys of earlier ones with the same value, as a log does
        keys[n - m:] = keys[_ranks(n - m, m, _gen(seed, 2), False)]
        keys = keys[torch.randperm(n, device=DEV, generator=_gen(seed, 3))]
    q, present = _queries(case, seed, keys)
    # which of a repeated key's pairs is the new one is the schedule's choice: a program that
    # loads such a log asks for no statuses
    st = dict(keys=keys, vals=_vals(keys), q=q, status=m == 0)
    if table:
        st["t"] = S.SlabHash(*_geometry(n, case["util"]), *_hash(seed))
    one = [torch.ones(n, dtype=torch.int64, device=DEV)] if m == 0 else []
    return st, lambda: (*one, *_found(q, present))


def _grow(case, seed, table):
    n = case["keys"]
    keys = _keys(seed, 0, n)
    size = -(-n // case["batches"])
    cut = [slice(i, min(n, i + size)) for i in range(0, n, size)]
    vals = _vals(keys)
    q, present = _queries(case, seed, keys)
    st = dict(keys=[keys[c] for c in cut], vals=[vals[c] for c in cut], q=q)
    if table:
        st["t"] = S.SlabHash(*_geometry(n, case["util"]), *_hash(seed))
    return st, lambda: ([torch.ones(k.numel(), dtype=torch.int64, device=DEV)
                         for k in st["keys"]], _found(q, present))


def _phased(case, seed, table):
    n, ko = case["keys"], case["keys_only"]
    keys = _keys(seed, 0, n)
    q, present = _queries(case, seed, keys)
    gone = n // 4
    st = dict(keys=keys, vals=None if ko else _vals(keys), q=q, gone=keys[:gone].clone())
    if table:
        b = case["buckets"]
        pool = A.pool_slabs_for(n, b, PAIRS[ko])
        st["t"] = S.SlabHash(b, pool, *_hash(seed), keys_only=ko)

    def expected():
        one = torch.ones(n, dtype=torch.int64, device=DEV)
        left = present & ~torch.isin(q, st["gone"])
        return one, _found(q, present, ko), one[:gone], _found(q, left, ko)
    return st, expected


def _mixed(case, seed, table):
    n, m = case["keys"], case["ops"]
    half = min(int(m * case["update"] / 2), n // 8)
    pairs = case["batches"] // 2
    keys = _keys(seed, 0, n)
    fresh = _keys(seed, n, pairs * half)
    g = _gen(seed, 4)
    batches, expect = [], []
    for i in range(pairs):
        x, y = fresh[i * half:(i + 1) * half], keys[i * half:(i + 1) * half]
        for ins, out in ((x, y), (y, x)):
            rest = m - 2 * half
            present = torch.rand(rest, device=DEV, generator=g) < 0.5
            at = pairs * half + _ranks(n - pairs * half, rest, g, False)
            k = torch.cat([ins, out, torch.where(present, keys[at], _keys(seed, 1 << 27, rest))])
            o = torch.cat([torch.full((half,), INSERT), torch.full((half,), DELETE),
                           torch.full((rest,), SEARCH)]).to(torch.uint8).to(DEV)
            ok = torch.cat([torch.ones(2 * half, dtype=torch.bool, device=DEV), present])
            p = torch.randperm(m, device=DEV, generator=g)
            k, o, ok = k[p], o[p], ok[p]
            v = _vals(k)
            batches.append((o, k, v))
            expect.append((torch.where((o == SEARCH) & ok, v, -1).to(torch.int64),
                           ok.to(torch.int64)))
    st = dict(batches=batches)
    if table:
        st["t"] = S.SlabHash(*_geometry(n, case["util"], 2 * pairs * half), *_hash(seed))
        _fill(st["t"], keys, _vals(keys))
    return st, lambda: expect


def _batched(case, seed, table):
    r = random.Random(seed * 31 + 5)
    T = case["tables"]

    def shares(total):  # log-uniform shares of a total, a factor of 16 between the extremes
        w = [math.exp(r.uniform(0, math.log(16))) for _ in range(T)]
        cut = [40 * i + int((total - 40 * T) * sum(w[:i]) / sum(w)) for i in range(T)] + [total]
        return [b - a for a, b in zip(cut, cut[1:])]

    ns, ls = shares(case["keys"]), shares(case["ops"])
    at, ops, keys, ok, params, fills = 0, [], [], [], [], []
    g = _gen(seed, 6)
    for n, m in zip(ns, ls):
        ins, gone = int(0.3 * m), min(int(0.1 * m), n // 4)
        rest = m - ins - gone
        u = _keys(seed, at, n + ins + rest)
        at += n + ins + rest
        present = torch.rand(rest, device=DEV, generator=g) < 0.5
        hits = u[gone + _ranks(n - gone, rest, g, False)]
        k = torch.cat([u[n:n + ins], u[:gone], torch.where(present, hits, u[n + ins:])])
        o = torch.zeros(m, dtype=torch.uint8, device=DEV)
        o[:ins], o[ins:ins + gone] = INSERT, DELETE
        one = torch.ones(ins + gone, dtype=torch.bool, device=DEV)
        p = torch.randperm(m, device=DEV, generator=g)
        keys.append(k[p])
        ops.append(o[p])
        ok.append(torch.cat([one, present])[p])
        b = max(1, int(n / (31 * 0.62)))
        params.append(S.ShParams(b, S.pool_slabs_bound(n + ins, 1), *_hash(seed + b)))
        fills.append(u[:n])
    ops, keys, ok = torch.cat(ops), torch.cat(keys), torch.cat(ok)
    vals = _vals(keys)
    st = dict(ops=ops, keys=keys, vals=vals, nb=T)
    if table:
        st["t"] = S.MultiSlabHash(params)
        for tb, u in zip(st["t"].tables, fills):
            tb.insert(u, _vals(u), status=False)
        off = [sum(ls[:i]) for i in range(T)]
        st["desc"] = torch.from_numpy(S.pack_batch_descs(off, ls, range(T))).to(DEV)
    return st, lambda: (torch.where((ops == SEARCH) & ok, vals, -1).to(torch.int64),
                        ok.to(torch.int64))


def _multiset(case, seed, table):
    n, c = case["keys"], case["copies"]
    keys = _keys(seed, 0, n)
    p = torch.randperm(n, device=DEV, generator=_gen(seed, 7))
    st = dict(keys=keys, vals=[_vals(keys, 77 * i) for i in range(c)], q=keys[p],
              gone=keys[:n // 2].clone())
    if table:
        st["t"] = S.SlabHash(*_geometry(n * c, case["util"]), *_hash(seed), duplicates=True)

    def expected():
        v = torch.stack([x[p] for x in st["vals"]], 1).to(torch.int64)
        left = p >= n // 2
        return ([torch.ones(n, dtype=torch.int64, device=DEV)] * c,
                (torch.full((n,), c, dtype=torch.int64, device=DEV),
                 torch.arange(n, dtype=torch.int64, device=DEV) * c, v.reshape(-1)),
                torch.full((n // 2,), c, dtype=torch.int64, device=DEV),
                (torch.where(left, v[:, 0], -1), left.to(torch.int64)))
    return st, expected


KINDS = dict(lookup=_lookup, build=_build, grow=_grow, phased=_phased, mixed=_mixed,
             batched=_batched, multiset=_multiset)


def prepare(case, seed):
    state, _ = KINDS[case["kind"]](case, seed, True)
    state["kind"] = case["kind"]
    return state


def exact(case, seed):
    return KINDS[case["kind"]](case, seed, False)[1]()


# --------------------------------------------------------------------------------------------
# The passes

def run(s):
    t, kind = s["t"], s["kind"]
    if kind == "lookup":
        return t.search(s["q"])
    if kind == "build":
        t.reset()
        st = t.build(s["keys"], s["vals"], status=s["status"])
        found = t.search(s["q"])
        return (st, *found) if s["status"] else found
    if kind == "grow":
        t.reset()
        return [t.insert(k, v) for k, v in zip(s["keys"], s["vals"])], t.search(s["q"])
    if kind == "phased":
        t.reset()
        st = t.build(s["keys"], s["vals"])
        before = t.search(s["q"])
        gone = t.delete(s["gone"])
        return st, before, gone, t.search(s["q"])
    if kind == "mixed":
        out = [t.mixed(o, k, v) for o, k, v in s["batches"]]
        t.flush()
        return out
    if kind == "batched":
        return t.mixed(s["desc"], s["nb"], s["ops"], s["keys"], s["vals"])
    t.reset()
    st = [t.insert(s["keys"], v) for v in s["vals"]]
    found = t.search_all(s["q"])
    gone = t.delete_all(s["gone"])
    return st, found, gone, t.search(s["q"])


def work(case):
    """Bytes a pass cannot do without: its inputs read, its outputs written, and each entry of
    the table that the pass has to see or set, once (8 bytes a pair, 4 a key)."""
    kind, n = case["kind"], case["keys"]
    if kind == "lookup":
        # every query needs its key's pair, or the keys of its bucket; no more than the table
        per_miss = 4 * 31 * case["util"]
        q = case["queries"]
        table = q * (8 * case["hit"] + per_miss * (1 - case["hit"]))
        return dict(bytes=9 * q + min(table, 8 * n), flops=0)
    if kind == "build":
        q = case["queries"]
        return dict(bytes=(8 + 8 + 1) * n + 9 * q + min(8 * n, 48 * q), flops=0)
    if kind == "grow":
        q = case["queries"]
        return dict(bytes=(8 + 8 + 1) * n + 9 * q + min(8 * n, 48 * q), flops=0)
    if kind == "phased":
        e, q = (4 if case["keys_only"] else 8), case["queries"]
        return dict(bytes=(2 * e + 1) * n + 2 * (9 * q + min(e * n, 48 * q)) + (n // 4) * (5 + 2 * e),
                    flops=0)
    if kind == "mixed":
        m = case["batches"] * case["ops"]
        return dict(bytes=m * (9 + 5 + 16) + 8 * n, flops=0)
    if kind == "batched":
        return dict(bytes=case["ops"] * (9 + 5 + 16), flops=0)
    c = case["copies"]
    return dict(bytes=n * c * (8 + 8 + 1) + n * (4 + 12 + 8 * c) + n // 2 * (8 + 16 * c) + 9 * n
                + 16 * n * c, flops=0)
