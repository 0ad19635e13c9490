"""GPU tests of sh_search_all_offsets where one block sums up the blocks' sums: many blocks."""
import pytest
import torch

from paper_1710_11246_amd import slabhash as S

pytestmark = pytest.mark.gpu
BLOCK = 8192   # counts per block of the kernels
DIRECT = 4096  # blocks whose sums each block adds up itself


# both sides of the line, and both sides of one turn of the summing block (8192 sums)
@pytest.mark.parametrize("blocks,more", [(DIRECT, 0), (DIRECT, 1), (2 * DIRECT, -1), (2 * DIRECT, 0),
                                         (2 * DIRECT, 1), (2 * DIRECT + 9, 3)])
def test_offsets_of_many_blocks(blocks, more):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = blocks * BLOCK + more
    c = torch.randint(-2**31, 2**31, (n,), dtype=torch.int64, device="cuda").to(torch.int32)
    off = torch.full((n,), -7, dtype=torch.int64, device="cuda")
    total = int(S.sh_search_all_offsets(c, off)[0])
    # counts are unsigned
    want = torch.cumsum(c.to(torch.int64) & 0xFFFFFFFF, 0)
    assert total == int(want[-1])
    assert int(off[0]) == 0 and bool((off[1:] == want[:-1]).all())
