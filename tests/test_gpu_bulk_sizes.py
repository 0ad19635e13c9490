"""GPU tests of the bulk form at its largest: parts made smaller, or taken in pieces, because their
slabs fill the LDS, and batches longer than one pass over the kernels."""
import sys

import pytest
import torch

from paper_1710_11246_amd import autotune as A
from paper_1710_11246_amd import slabhash as S

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S.lib()


def work_for(t, kind, n):
    nb = S.sh_bulk_bytes(t.handle, kind, n)
    assert nb > 0
    return torch.full((nb,), 0xA5, dtype=torch.uint8, device="cuda")


# 16 operations per bucket at 2^25 (smaller parts); the most buckets whose slabs fit at 2^26 (a
# queue shorter than a part); one batch of two passes, the second a tile and a bit
@pytest.mark.parametrize("n,B", [(1 << 25, 1 << 21), (1 << 26, 6_600_000),
                                 ((1 << 26) + 32771, 3_900_007)])
@pytest.mark.parametrize("keys_only", [False, True])
def test_largest(n, B, keys_only):
    say("case: bulk form, large", n, B, keys_only)
    t = S.SlabHash(B, A.pool_slabs_for(n, B), 1234567, 89, keys_only=keys_only)
    cs = torch.cuda.current_stream().cuda_stream
    # every key from 0 up: a multiplicative hash spreads them; values tell the key
    k = torch.arange(n, dtype=torch.int32, device="cuda")
    lib = S.lib()
    if keys_only:
        t.insert(k, None, status=False)
        want = k
    else:
        w = work_for(t, S.SH_OP_INSERT, n)
        st = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
        assert lib.sh_insert_bulk(t.handle, k.data_ptr(), (~k).contiguous().data_ptr(), n,
                                  st.data_ptr(), w.data_ptr(), w.numel(), cs) == S.SH_OK
        assert bool((st == 1).all())
        s = t.stats()
        assert s["live"] == n and s["violations"] == 0 and s["error_word"] == 0
        want = ~k
    q = k + n // 2  # half of them absent
    w = work_for(t, S.SH_OP_SEARCH, n)
    v = torch.full((n,), 7, dtype=torch.int32, device="cuda")
    f = torch.full((n,), 9, dtype=torch.uint8, device="cuda")
    assert lib.sh_search_bulk(t.handle, q.data_ptr(), n, v.data_ptr(), f.data_ptr(), w.data_ptr(),
                              w.numel(), cs) == S.SH_OK
    there = q < n
    assert bool((f == there).all())
    assert bool((v == torch.where(there, want[(q % n).long()], -1)).all())
