"""GPU tests of sh_search_all_offsets: the exclusive prefix sums of SEARCHALL counts."""
import numpy as np
import pytest
import torch

from paper_1710_11246_amd import slabhash as S

pytestmark = pytest.mark.gpu
BLOCK = 8192  # counts per block of the kernels


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S.lib()


# one thread's counts, one block's and their neighbours, and more blocks than a block has threads
@pytest.mark.parametrize("n", [0, 1, 7, 8, 9, BLOCK - 1, BLOCK, BLOCK + 1, 3 * BLOCK + 5, 1000003,
                               1025 * BLOCK + 3])
@pytest.mark.parametrize("top", [5, 1 << 32])
def test_offsets(n, top):
    rng = np.random.default_rng(n + top)
    c = rng.integers(0, top, n + 1, dtype=np.uint64).astype(np.uint32)
    d = S.to_dev(c)[1:]  # an odd word address
    for counts in (d, d.clone()):
        off = torch.full((n,), -7, dtype=torch.int64, device="cuda")
        total = int(S.sh_search_all_offsets(counts, off)[0])
        want = np.concatenate([np.zeros(1, np.uint64), np.cumsum(c[1:].astype(np.uint64))])
        assert total == int(want[-1])
        assert (off.cpu().numpy().astype(np.uint64) == want[:-1]).all()


def test_refused():
    lib = S.lib()
    w = torch.zeros(4, dtype=torch.int64, device="cuda")
    p = w.data_ptr()
    assert lib.sh_search_all_offsets(p, 1 << 32, p, p, None) == S.SH_EINVAL
    assert lib.sh_search_all_offsets(None, 4, p, p, None) == S.SH_EINVAL
    assert lib.sh_search_all_offsets(p, 4, None, p, None) == S.SH_EINVAL
    assert lib.sh_search_all_offsets(p, 4, p, None, None) == S.SH_EINVAL
    assert lib.sh_search_all_offsets(p, 4, p + 4, p, None) == S.SH_EINVAL
    assert S.lib().sh_offsets_words(BLOCK + 1) == 3


@pytest.mark.parametrize("where", ["current", "other", "number"])
def test_search_all_on_streams(where):
    t = S.SlabHash(64, 2048 * 4, 12345, 678, duplicates=True)
    k = torch.arange(1000, dtype=torch.int32, device="cuda") % 300
    t.insert(k, torch.arange(1000, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    q = torch.arange(400, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    c, o, v = t.search_all(q, stream={"current": None, "other": s, "number": s.cuda_stream}[where])
    torch.cuda.synchronize()
    want = [sorted(range(i, 1000, 300)) if i < 300 else [] for i in range(400)]
    assert c.tolist() == [len(w) for w in want]
    for i in range(400):
        assert sorted(v[o[i]:o[i] + c[i]].tolist()) == want[i]
