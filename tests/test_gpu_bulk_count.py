"""GPU tests of what a table's choice of form counts: calls since the last reset that has run."""
import pytest
import torch

from paper_1710_11246_amd import slabhash as S

pytestmark = pytest.mark.gpu
N, B = 1 << 20, 50000


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S.lib()


def forms(t):
    """Whether an insert of N more has a bulk form, and whether the binding would take it."""
    return (S.sh_bulk_bytes(t.handle, S.SH_OP_INSERT, N) > 0,
            S.sh_bulk_choice(t.handle, S.SH_OP_INSERT, N) > 0)


def test_a_captured_reset_has_not_run():
    t = S.SlabHash(B, S.pool_slabs_bound(2 * N), 12345, 678)
    k = torch.arange(N, dtype=torch.int32, device="cuda")
    assert forms(t) == (True, True)
    t.insert(k, k, status=False)
    assert forms(t) == (False, False)  # 42 per bucket
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    S.sh_capture_begin(s)
    S.sh_reset(t.handle, s)
    g = S.sh_capture_end(s)
    assert forms(t) == (False, False)
    # the captured reset runs: the table is empty, which the count does not know
    S.sh_graph_launch(g, s)
    torch.cuda.synchronize()
    assert t.stats()["live"] == 0 and forms(t) == (False, False)
    st = t.insert(k, k)
    assert bool((st == 1).all())
    S.sh_graph_destroy(g)
    t.reset()
    assert forms(t) == (True, True)


def test_what_is_counted():
    """Replacing inserts and mixed batches count like new pairs; deletes and searches do not."""
    t = S.SlabHash(B, S.pool_slabs_bound(2 * N), 12345, 678)
    k = torch.arange(1000, dtype=torch.int32, device="cuda")
    t.search(k)
    t.delete(k)
    assert forms(t) == (True, True)
    t.insert(k, k)
    assert forms(t) == (True, True)  # 20 per bucket, beside some held
    few = S.SlabHash(N // 8, S.pool_slabs_bound(2 * N), 12345, 678)  # 8 per bucket
    assert forms(few) == (True, True)
    few.mixed(torch.zeros(1000, dtype=torch.uint8, device="cuda"), k, k)
    assert forms(few) == (True, False)
    few.reset()
    few.insert(k, k)
    few.insert(k, k)
    assert forms(few) == (True, False)
