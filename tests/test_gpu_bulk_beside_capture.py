"""GPU tests of large calls on one stream while another stream is being captured: the capture goes
on, the call answers, and the captured work replays."""
import sys
import threading

import pytest
import torch

from paper_1710_11246_amd import slabhash as S

pytestmark = pytest.mark.gpu
N = 1 << 22


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    S.lib()


@pytest.mark.parametrize("who", ["torch graph, this thread", "torch graph, another thread",
                                 "library capture, this thread"])
def test_large_calls_beside_a_capture(who):
    say("case: large calls beside a capture:", who)
    t = S.SlabHash(100003, S.pool_slabs_bound(N), 12345, 678)
    k = torch.arange(N, dtype=torch.int32, device="cuda")
    t.insert(k, ~k, status=False)
    x = torch.zeros(1024, dtype=torch.int32, device="cuda")
    v, f = torch.zeros_like(k), torch.zeros(N, dtype=torch.uint8, device="cuda")
    few = torch.zeros(1024, dtype=torch.int32, device="cuda")
    captured, call = torch.cuda.Stream(), torch.cuda.Stream()
    assert S.sh_bulk_choice(t.handle, S.SH_OP_SEARCH, N, call) > 0
    torch.cuda.synchronize()
    torch.cuda.empty_cache()  # the call's workspace has to come from the device
    errors = []

    def large_call():
        try:
            S.sh_search(t.handle, k, v, f, call)
        except Exception as e:  # reported below, by the test's own thread
            errors.append(e)

    if who.startswith("torch"):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=captured):
            x.add_(1)
            if "another" in who:
                th = threading.Thread(target=large_call)
                th.start()
                th.join()
            else:
                large_call()
            S.sh_search(t.handle, k[:1024], few, None, captured)
        replay, end = g.replay, lambda: None
    else:
        S.sh_capture_begin(captured)
        S.sh_search(t.handle, k[:1024], few, None, captured)
        large_call()
        with torch.cuda.stream(captured):
            x.add_(1)
        h = S.sh_capture_end(captured)
        replay, end = (lambda: S.sh_graph_launch(h, captured)), (lambda: S.sh_graph_destroy(h))
    assert not errors, errors
    torch.cuda.synchronize()
    assert bool((v == ~k).all()) and bool((f == 1).all())
    for i in range(3):
        few.zero_()
        torch.cuda.synchronize()
        replay()
        torch.cuda.synchronize()
        assert bool((few == ~k[:1024]).all()) and bool((x == i + 1).all())
        t.search(k)  # eager work between the replays
    end()
