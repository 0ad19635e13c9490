"""What the Python binding does around a call (CPU, with the library stood in for)."""
import pytest
import torch

from paper_1710_11246_amd import slabhash as S


class Library:
    """Answers how large a workspace is, and counts the questions and the changes of the thread's
    capture mode."""

    def __init__(self, nbytes):
        self.nbytes, self.asked, self.modes = nbytes, [], []

    def sh_bulk_choice(self, t, kind, n, stream):
        self.asked.append((kind, n, stream))
        return self.nbytes

    def hipThreadExchangeStreamCaptureMode(self, mode):
        self.modes.append(mode._obj.value)
        mode._obj.value = 0
        return 0


@pytest.mark.parametrize("kind,n", [(S.SH_OP_SEARCH, 7 << 19), (S.SH_OP_INSERT, 1 << 17)])
def test_a_call_without_a_bulk_form_builds_no_stream_object(monkeypatch, kind, n):
    """Large enough to ask, refused by the library: one question, by the stream's number."""
    def no(*a, **k):
        raise AssertionError("a Stream object for a call that does not need it")

    fake = Library(0)
    monkeypatch.setattr(S, "lib", lambda: fake)
    monkeypatch.setattr(S, "_current_stream", lambda: 7)
    monkeypatch.setattr(torch.cuda, "current_stream", no)
    monkeypatch.setattr(torch.cuda, "stream", no)
    keys = torch.empty(n, dtype=torch.int32)
    assert S._bulk_work(None, kind, keys, None) is None
    assert S._bulk_work(None, kind, keys, 9) is None
    assert fake.asked == [(kind, n, 7), (kind, n, 9)]
    assert S._bulk_work(None, kind, keys[1:], None) is None  # below the line: not even asked
    assert len(fake.asked) == 2 and not fake.modes


def test_a_call_on_the_current_stream_builds_no_stream_object(monkeypatch):
    """Its workspace is the current stream's; the thread's capture mode is relaxed for the
    allocation and set back."""
    def no(*a, **k):
        raise AssertionError("a Stream object for the current stream")

    fake = Library(1000)
    monkeypatch.setattr(S, "lib", lambda: fake)
    monkeypatch.setattr(S, "_current_stream", lambda: 7)
    monkeypatch.setattr(torch.cuda, "current_stream", no)
    monkeypatch.setattr(torch.cuda, "stream", no)
    keys = torch.empty(1 << 17, dtype=torch.int32)
    for stream in (None, 7):
        fake.modes.clear()
        assert S._bulk_work(None, S.SH_OP_INSERT, keys, stream).numel() == 1000
        assert fake.modes == [2, 0]
    assert S._bulk_work(None, S.SH_OP_INSERT, keys, 9) is None  # of an owner unknown to torch

    def full(*a, **k):
        raise torch.cuda.OutOfMemoryError("no room")

    fake.modes.clear()
    monkeypatch.setattr(torch, "empty", full)
    assert S._bulk_work(None, S.SH_OP_INSERT, keys, None) is None and fake.modes == [2, 0]
