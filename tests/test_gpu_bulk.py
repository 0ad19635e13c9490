"""GPU tests of the bulk form (sh_search_bulk, sh_insert_bulk): batches split by bucket range give
what the plain calls and the oracle give, at the edges of tiles and pieces, in every table mode,
on long lists, with repeated and reserved keys, and beside calls on other streams."""
import ctypes
import sys

import numpy as np
import pytest
import torch

from paper_1710_11246_amd import slabhash as S
from paper_1710_11246_amd import workload as W

import host_walk as HW
from test_gpu_parity import assert_same_table

pytestmark = pytest.mark.gpu
M = S.SH_SLAB_PAIRS
SMALLEST = {S.SH_OP_SEARCH: 3 << 20, S.SH_OP_INSERT: 1 << 17}


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S.lib()


def bulk_search(t, q, found=True):
    """The bulk call itself, with a workspace of its own; fails if there is no bulk form."""
    n = q.numel()
    nb = S.sh_bulk_bytes(t.handle, S.SH_OP_SEARCH, n)
    assert nb > 0
    work = torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")
    v = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    f = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    code = S.lib().sh_search_bulk(t.handle, q.data_ptr(), n, v.data_ptr(),
                                  f.data_ptr() if found else None, work.data_ptr(), nb,
                                  torch.cuda.current_stream().cuda_stream)
    assert code == S.SH_OK
    return v, f


def plain_search(t, q):
    n = q.numel()
    v = torch.empty(n, dtype=torch.int32, device="cuda")
    f = torch.empty(n, dtype=torch.uint8, device="cuda")
    assert S.lib().sh_search(t.handle, q.data_ptr(), n, v.data_ptr(), f.data_ptr(),
                             torch.cuda.current_stream().cuda_stream) == S.SH_OK
    return v, f


def bulk_insert(t, k, v, status=True):
    n = k.numel()
    nb = S.sh_bulk_bytes(t.handle, S.SH_OP_INSERT, n)
    assert nb > 0
    work = torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")
    st = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    code = S.lib().sh_insert_bulk(t.handle, k.data_ptr(), v.data_ptr(), n,
                                  st.data_ptr() if status else None, work.data_ptr(), nb,
                                  torch.cuda.current_stream().cuda_stream)
    assert code == S.SH_OK
    return st


def same(a, b):
    return bool((a[0] == b[0]).all()) and bool((a[1] == b[1]).all())


def table(seed, n, B, **mode):
    rng = W.SplitMix64(seed)
    a, b = W.hash_params(rng, S.SH_HASH_PRIME)
    return S.SlabHash(B, S.pool_slabs_bound(2 * n), a, b, **mode), a, b


# the smallest batch; around a whole tile of 8192 and of 16384 and the line where the tile grows
# (3 * 2^20); buckets from one per part up to the line of six operations each
@pytest.mark.parametrize("n,B", [(1 << 21, 54343), ((3 << 20) + 1, 1024), ((3 << 20) + 8191, 4096),
                                 (3 << 20, 100003), ((3 << 20) + 1, 100003),
                                 ((3 << 20) + 16383, 500000), (2300003, 300007)])
@pytest.mark.parametrize("mode", ["pairs", "duplicates", "keys_only", "both"])
def test_search(n, B, mode):
    say("case: bulk search", n, B, mode)
    kw = dict(duplicates=mode in ("duplicates", "both"), keys_only=mode in ("keys_only", "both"))
    t, _, _ = table(31 + B, 1 << 21, B, **kw)
    keys = torch.from_numpy(W.distinct_keys(5, 0, n).view(np.int32)).cuda()
    held = keys[:n // 2]
    vals = held ^ 0x1234567
    t.insert(held, None if kw["keys_only"] else vals)
    if kw["duplicates"]:
        t.insert(held[: n // 8], None if kw["keys_only"] else ~vals[: n // 8])
    t.delete(held[: n // 64])
    q = keys.clone()
    q[3::997] = -1  # reserved
    q[5::1009] = -2  # reserved where slabs hold keys alone
    v, f = bulk_search(t, q)
    assert same((v, f), plain_search(t, q))
    assert bool((f[q == -1] == 0).all()) and bool((v[q == -1] == -1).all())
    assert t.stats()["error_word"] & S.SH_ERR_RESERVED_KEY
    v2, _ = bulk_search(t, q, found=False)
    assert bool((v2 == v).all())
    # keys and outputs at odd word addresses
    x = torch.empty(n + 1, dtype=torch.int32, device="cuda")
    x[1:] = q
    assert same(bulk_search(t, x[1:]), (v, f))


def test_search_long_lists_and_popular_keys():
    """Lists of about eight slabs; batches of one key, of few keys and of Zipf ranks."""
    say("case: bulk search, long lists and popular keys")
    n, B = 3 << 20, 12288
    t, _, _ = table(77, n, B)
    keys = torch.from_numpy(W.distinct_keys(9, 0, n).view(np.int32)).cuda()
    t.insert(keys, ~keys)
    absent = torch.from_numpy(W.distinct_keys(9, n, n).view(np.int32)).cuda()
    ranks = torch.from_numpy(W.zipf_ranks(W.SplitMix64(3), n, n, 1.1) - 1).cuda()
    few = torch.arange(n, device="cuda") % 5
    batches = [keys, absent, torch.cat([keys[: n // 2], absent[: n // 2 + 7]]), keys[ranks],
               keys[few], keys[:1].expand(n).contiguous(), absent[:1].expand(n).contiguous(),
               torch.where(few == 0, keys[ranks], absent[few])]
    for i, q in enumerate(batches):
        assert same(bulk_search(t, q), plain_search(t, q)), i


# the smallest batch, the fewest inserts per bucket and a full base slab's worth of them, and both
# sides of the line where the tile grows; tables with room for a second batch and without
@pytest.mark.parametrize("n,B", [(1 << 17, 5043), ((1 << 17) + 1, 21845), (700001, 60013),
                                 (3 << 19, 78643), ((3 << 19) + 5, 150001), (1 << 19, 20200)])
def test_insert(oracle_mod, n, B):
    """Fresh keys, the same keys with new values, and a batch with repeated, present, fresh and
    reserved keys: statuses, values and the whole structure against the oracle."""
    say("case: bulk insert", n, B)
    t, a, b = table(13 + n, n, B)
    o = oracle_mod.Oracle(B, M, a, b)
    all_keys = W.distinct_keys(17, 0, 2 * n)
    k, v = all_keys[:n], W.value_of(all_keys[:n])
    st = bulk_insert(t, S.to_dev(k), S.to_dev(v))
    assert bool((st == 1).all())
    o.replace(k, v)
    assert_same_table(t, o)
    t2, _, _ = table(13 + n, n, B)  # the same table again: no statuses asked for
    bulk_insert(t2, S.to_dev(k), S.to_dev(v), status=False)
    assert_same_table(t2, o)
    # a second batch on the filled table: the first half of the keys with new values, repeats of
    # the fresh ones, reserved keys
    if 2 * n > 26 * B:
        return
    k2 = np.concatenate([k[: n // 2], all_keys[n:n + n // 4], all_keys[n:n + n // 4],
                         all_keys[n:n + n - 2 * (n // 4) - n // 2]]).astype(np.uint32)
    k2 = k2[W.SplitMix64(8).permutation(k2.size)]
    k2[7::5003] = 0xFFFFFFFF
    v2 = np.arange(k2.size, dtype=np.uint32)
    st = bulk_insert(t, S.to_dev(k2), S.to_dev(v2)).cpu().numpy()
    ok = k2 != 0xFFFFFFFF
    assert (st[~ok] == 0).all() and t.stats()["error_word"] == S.SH_ERR_RESERVED_KEY
    # per key: a present key's inserts all replace; of a fresh key's exactly one is new, and the
    # table holds the value of one of the batch's inserts: with several, not only the new one's
    uk, inv, cnt = np.unique(k2[ok], return_inverse=True, return_counts=True)
    new = np.bincount(inv, weights=(st[ok] == 1)).astype(int)
    assert set(np.unique(st[ok])) <= {1, 2}
    assert (new == ~np.isin(uk, k)).all()
    got, f = plain_search(t, S.to_dev(uk))
    got = S.to_host_u32(got)
    assert bool((f == 1).all()) and (k2[got] == uk).all()
    several = (cnt > 1) & (new == 1)
    assert (st[got[several]] == 2).all()
    o.replace(uk, got)
    assert_same_table(t, o)


@pytest.mark.parametrize("pool_blocks", [64, 4])
def test_insert_leaves_full_slabs_to_the_plain_kernel(oracle_mod, pool_blocks):
    """A bulk batch into a table whose base slabs are mostly full: its inserts go down the lists,
    and a pool too small fails some of them. (A graph's replay fills the table: the host does not
    count its inserts, so the bulk form is still chosen.)"""
    say("case: bulk insert into full base slabs", pool_blocks)
    B, n = 20200, 1 << 19
    keys = W.distinct_keys(23, 0, 2 * n)
    rng = W.SplitMix64(99)
    a, b = W.hash_params(rng, S.SH_HASH_PRIME)
    t = S.SlabHash(B, 2048 * pool_blocks, a, b)
    k0, k1 = S.to_dev(keys[:n]), S.to_dev(keys[n:])
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    S.sh_capture_begin(s)
    S.sh_insert(t.handle, k0, k0, None, s)
    g = S.sh_capture_end(s)
    t.reset()
    torch.cuda.synchronize()
    S.sh_graph_launch(g, s)
    torch.cuda.synchronize()
    S.sh_graph_destroy(g)
    before = t.stats()["live"]
    st = bulk_insert(t, k1, k1)
    s1 = t.stats()
    bad = int((st == 0).sum())
    assert int((st == 1).sum()) == n - bad == s1["live"] - before and s1["violations"] == 0
    v, f = plain_search(t, k1)
    assert bool((f == (st == 1)).all()) and bool((v == torch.where(st == 1, k1, -1)).all())
    if pool_blocks == 64:
        assert bad == 0 and before == n and s1["error_word"] == 0
        o = oracle_mod.Oracle(B, M, a, b)
        for k in (keys[:n], keys[n:]):
            o.replace(k, k)
        assert_same_table(t, o)
    else:
        assert bad > 0 and s1["error_word"] == S.SH_ERR_POOL_EXHAUSTED


@pytest.mark.parametrize("B,bulks", [(41000, 2), (20200, 1)])
def test_bulk_and_plain_inserts_at_once(B, bulks):
    """Two streams insert the same keys while a third inserts half of them in small plain batches:
    one insert of each key is new, every other replaces, no key enters twice. 13 keys a bucket
    with both streams' inserts in the bulk form, and 26, so that lists grow, with one's."""
    say("case: bulk and plain inserts on three streams", B)
    n = 1 << 19
    t, _, _ = table(5, n, B)
    k = torch.from_numpy(W.distinct_keys(29, 0, n).view(np.int32)).cuda()
    perm = torch.randperm(n, device="cuda")
    sets = [(k, k ^ 1), (k[perm], k[perm] ^ 2)]
    part = (k[: n // 2].flip(0).contiguous(), k[: n // 2].flip(0).contiguous() ^ 3)
    for rep in range(3):
        t.reset()
        nb = S.sh_bulk_bytes(t.handle, S.SH_OP_INSERT, n)
        assert nb
        works = [torch.empty(nb, dtype=torch.uint8, device="cuda") for _ in sets]
        sts = [torch.full((n,), 9, dtype=torch.uint8, device="cuda") for _ in sets]
        st3 = torch.full((n // 2,), 9, dtype=torch.uint8, device="cuda")
        ss = [torch.cuda.Stream() for _ in range(3)]
        torch.cuda.synchronize()
        done = 0
        for (kk, vv), w, st, s in zip(sets, works, sts, ss):
            done += S.sh_bulk_bytes(t.handle, S.SH_OP_INSERT, n) > 0
            code = S.lib().sh_insert_bulk(t.handle, kk.data_ptr(), vv.data_ptr(), n,
                                          st.data_ptr(), w.data_ptr(), nb, s.cuda_stream)
            assert code == S.SH_OK
        for i in range(0, n // 2, 1 << 15):
            S.sh_insert(t.handle, part[0][i:i + (1 << 15)], part[1][i:i + (1 << 15)],
                        st3[i:i + (1 << 15)], ss[2])
        torch.cuda.synchronize()
        assert done == bulks
        s1 = t.stats()
        assert s1["live"] == n and s1["violations"] == 0 and s1["error_word"] == 0
        new = torch.zeros(n, dtype=torch.int32, device="cuda")
        new += (sts[0] == 1).int()
        new[perm] += (sts[1] == 1).int()
        new[: n // 2] += (st3.flip(0) == 1).int()
        assert bool((new == 1).all())
        for st in (*sts, st3):
            assert bool(((st == 1) | (st == 2)).all())
        v, f = plain_search(t, k)
        d = v ^ k
        ok = (d == 1) | (d == 2)
        ok[: n // 2] |= d[: n // 2] == 3
        assert bool((f == 1).all()) and bool(ok.all())
        HW.check_structure(t)


def test_where_the_plain_form_serves():
    """Calls that keep the plain form, and arguments that are refused."""
    say("case: bulk form's lines")
    t, _, _ = table(3, 1 << 21, 20000)
    for kind, least in SMALLEST.items():
        assert S.sh_bulk_bytes(t.handle, kind, least) > 0
        assert S.sh_bulk_bytes(t.handle, kind, least - 1) == 0
        assert S.sh_bulk_bytes(t.handle, kind, 0) == 0
    for kind in (S.SH_OP_DELETE, S.SH_KIND_MIXED, 17):
        assert S.sh_bulk_bytes(t.handle, kind, 1 << 21) == 0
    big, _, _ = table(3, 1 << 10, 1 << 15)  # more than the caches hold
    assert S.sh_bulk_bytes(big.handle, S.SH_OP_SEARCH, 1 << 21) > 0
    assert S.sh_bulk_bytes(big.handle, S.SH_OP_SEARCH, (1 << 21) - 1) == 0
    wide, _, _ = table(3, 1 << 10, (1 << 21) // 6 + 1)  # fewer than six per bucket
    assert S.sh_bulk_bytes(wide.handle, S.SH_OP_SEARCH, 1 << 21) == 0
    few, _, _ = table(3, 1 << 20, 1023)
    assert S.sh_bulk_bytes(few.handle, S.SH_OP_SEARCH, 3 << 20) == 0
    assert S.sh_bulk_bytes(t.handle, S.SH_OP_INSERT, 26 * 20000 + 1) == 0
    flagged, _, _ = table(3, 1 << 10, 20000, keys_only=True)
    assert S.sh_bulk_bytes(flagged.handle, S.SH_OP_INSERT, 1 << 20) == 0
    assert S.sh_bulk_bytes(flagged.handle, S.SH_OP_SEARCH, 3 << 20) > 0
    t.set_launch(16, 32)
    assert S.sh_bulk_bytes(t.handle, S.SH_OP_SEARCH, 3 << 20) == 0
    t.set_launch(0, 0, S.SH_LAUNCH_COUNTERS)
    assert S.sh_bulk_bytes(t.handle, S.SH_OP_SEARCH, 3 << 20) == 0
    t.set_launch()
    n = 3 << 20
    k = torch.from_numpy(W.distinct_keys(41, 0, n).view(np.int32)).cuda()
    t.insert(k, ~k)
    v = torch.empty(n, dtype=torch.int32, device="cuda")
    nb = S.sh_bulk_bytes(t.handle, S.SH_OP_SEARCH, n)
    work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    call = S.lib().sh_search_bulk
    assert call(t.handle, k.data_ptr(), n, v.data_ptr(), None, work.data_ptr() + 4, nb, None) == \
        S.SH_EINVAL
    assert call(None, k.data_ptr(), n, v.data_ptr(), None, work.data_ptr(), nb, None) == S.SH_EINVAL
    assert call(t.handle, None, n, v.data_ptr(), None, work.data_ptr(), nb, None) == S.SH_EINVAL
    assert call(t.handle, k.data_ptr(), n, None, None, work.data_ptr(), nb, None) == S.SH_EINVAL
    assert call(t.handle, k.data_ptr(), 1 << 32, v.data_ptr(), None, work.data_ptr(), nb, None) == \
        S.SH_EINVAL
    assert call(t.handle, k.data_ptr(), 0, v.data_ptr(), None, work.data_ptr(), nb, None) == S.SH_OK
    # without a workspace, or with one too small, the plain form answers
    for w, b in ((None, 0), (work.data_ptr(), nb - 1)):
        v.zero_()
        assert call(t.handle, k.data_ptr(), n, v.data_ptr(), None, w, b, None) == S.SH_OK
        torch.cuda.synchronize()
        assert bool((v == ~k).all())
    # a capturing stream: no bulk form, and the captured call replays
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    S.sh_capture_begin(s)
    assert S.sh_bulk_bytes(t.handle, S.SH_OP_SEARCH, n, s) == 0
    S.sh_search(t.handle, k, v, None, s)
    g = S.sh_capture_end(s)
    for _ in range(3):
        v.zero_()
        torch.cuda.synchronize()
        S.sh_graph_launch(g, s)
        torch.cuda.synchronize()
        assert bool((v == ~k).all())
    S.sh_graph_destroy(g)
    # another stream of torch's, and a stream of another owner (by its number)
    for other in (s, s.cuda_stream):
        v.zero_()
        torch.cuda.synchronize()
        S.sh_search(t.handle, k, v, None, other)
        torch.cuda.synchronize()
        assert bool((v == ~k).all())
    assert ctypes.sizeof(ctypes.c_size_t) == 8


@pytest.mark.parametrize("n,B", [((3 << 20) + 3, 100003), ((1 << 23) + 1, 300007)])
def test_values_of_all_ones_are_found(n, B):
    """A value that looks like an absent key's result: the flag alone tells them apart, in whole
    groups of four and in a last one."""
    say("case: bulk search, values all ones", n, B)
    t, _, _ = table(41, n, B)
    keys = torch.from_numpy(W.distinct_keys(43, 0, n).view(np.int32)).cuda()
    held = torch.arange(n, device="cuda") % 3 != 1
    vals = torch.where(torch.arange(n, device="cuda") % 2 == 0, -1, 7).to(torch.int32)
    t.insert(keys[held], vals[held], status=False)
    v, f = bulk_search(t, keys)
    assert bool((f == held).all())
    assert bool((v == torch.where(held, vals, -1)).all())
