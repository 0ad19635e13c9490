"""GPU tests of bulk inserts that repeat keys: every insert of a part larger than its queue, of a
bucket's line that overflows, and of keys that share a place, against the oracle."""
import sys

import numpy as np
import pytest
import torch

from paper_1710_11246_amd import slabhash as S
from paper_1710_11246_amd import workload as W

from test_gpu_parity import assert_same_table

pytestmark = pytest.mark.gpu
M = S.SH_SLAB_PAIRS


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S.lib()


def ranks(dist, n):
    """Which of n keys each of n inserts has."""
    i = np.arange(n)
    if dist == "one":
        return i * 0
    if dist == "five":
        return i % 5
    if dist == "twice":
        return W.SplitMix64(4).permutation(n) // 2
    if dist == "zipf":
        return W.zipf_ranks(W.SplitMix64(3), n, n, 1.1) - 1
    # one key's inserts make its part just longer than one queue (about 2,400 operations), than
    # four, and a bucket's line (32 places) full of it
    few = {"over one queue": 1500, "over four queues": 9000, "over one line": 40}[dist]
    return np.where(i % (n // few) == 0, 0, i)


def insert(t, k, v):
    """The bulk call with a workspace of its own: statuses, and how many inserts it listed for
    the plain kernel (the workspace's first word)."""
    n = k.size
    nb = S.sh_bulk_bytes(t.handle, S.SH_OP_INSERT, n)
    assert nb > 0
    dk, dv = S.to_dev(k), S.to_dev(v)
    work = torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")
    st = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    assert S.lib().sh_insert_bulk(t.handle, dk.data_ptr(), dv.data_ptr(), n, st.data_ptr(),
                                  work.data_ptr(), nb,
                                  torch.cuda.current_stream().cuda_stream) == S.SH_OK
    return st.cpu().numpy(), int(work[:4].cpu().numpy().view(np.uint32)[0])


def check(t, o, present, k, v, st):
    """One insert of a fresh key is new, every other replaces; the table holds the value of one of
    the key's inserts, with several not the new one's."""
    uk, inv, cnt = np.unique(k, return_inverse=True, return_counts=True)
    assert set(np.unique(st)) <= {1, 2}
    new = np.bincount(inv, weights=(st == 1)).astype(int)
    assert (new == ~np.isin(uk, present)).all()
    got, f = t.search(S.to_dev(uk))
    got = S.to_host_u32(got)
    assert bool((f == 1).all())
    at = got - v[0]  # values are v[0] + the insert's number
    assert (k[at] == uk).all()
    assert (st[at[(cnt > 1) & (new == 1)]] == 2).all()
    o.replace(uk, got)
    assert_same_table(t, o)


@pytest.mark.parametrize("dist", ["one", "five", "twice", "zipf", "over one line",
                                  "over one queue", "over four queues"])
@pytest.mark.parametrize("n,B", [(1 << 19, 43691), ((1 << 19) + 3, 26001)])
def test_repeated_keys(oracle_mod, dist, n, B):
    say("case: bulk insert of repeated keys", dist, n, B)
    a, b = W.hash_params(W.SplitMix64(B), S.SH_HASH_PRIME)
    t = S.SlabHash(B, S.pool_slabs_bound(2 * n), a, b)
    o = oracle_mod.Oracle(B, M, a, b)
    keys = W.distinct_keys(19, 0, n)
    k = keys[ranks(dist, n)]
    v = np.arange(n, dtype=np.uint32) + np.uint32(5)
    st, listed = insert(t, k, v)
    check(t, o, k[:0], k, v, st)
    # Listed are the lines' overflows of keys that share no place: the other keys of the buckets
    # of popular ones. (Both batches of 12 and of 20 per bucket; half of a Zipf batch's inserts are
    # of some 1300 keys with more than 20 each, whose buckets hold a few in a hundred.)
    assert listed <= n // 16
    if dist in ("one", "five"):
        assert listed == 0
    # the keys again, all present now, then half of them and fresh ones
    if 2 * n <= 26 * B:
        v = v + np.uint32(n)
        st, _ = insert(t, k, v)
        check(t, o, k, k, v, st)
        assert (st == 2).all()


def test_repeats_on_full_slabs(oracle_mod):
    """Popular keys whose buckets' base slabs are full: what the line shares goes to the plain
    kernel, or to a new slab, with the place it shares."""
    n, B = 1 << 19, 21000
    say("case: bulk insert of repeated keys into full slabs", n, B)
    a, b = W.hash_params(W.SplitMix64(5), S.SH_HASH_PRIME)
    t = S.SlabHash(B, S.pool_slabs_bound(4 * n), a, b)
    o = oracle_mod.Oracle(B, M, a, b)
    keys = W.distinct_keys(21, 0, 3 * n)
    v = np.arange(n, dtype=np.uint32)
    # 19 to 31 pairs a bucket before, by calls whose inserts the library does not count
    held = keys[:n]
    dk = S.to_dev(held)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    S.sh_capture_begin(s)
    S.sh_insert(t.handle, dk, dk, None, s)
    g = S.sh_capture_end(s)
    t.reset()
    torch.cuda.synchronize()
    S.sh_graph_launch(g, s)
    torch.cuda.synchronize()
    S.sh_graph_destroy(g)
    o.replace(held, held)
    r = ranks("zipf", n)
    k = np.where(np.arange(n) % 3 == 0, held[r], keys[n:][r + (np.arange(n) % 2)])
    st, _ = insert(t, k, v)
    check(t, o, held, k, v, st)
