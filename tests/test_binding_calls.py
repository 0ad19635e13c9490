"""What the Python binding does around a call (CPU, with the library stood in for)."""
import pytest
import torch

from paper_1710_11246_amd import slabhash as S


class Library:
    """Answers that no call has a bulk form, and counts the questions."""

    def __init__(self):
        self.asked = []

    def sh_bulk_choice(self, t, kind, n, stream):
        self.asked.append((kind, n, stream))
        return 0


@pytest.mark.parametrize("kind,n", [(S.SH_OP_SEARCH, 7 << 19), (S.SH_OP_INSERT, 1 << 17)])
def test_a_call_without_a_bulk_form_builds_no_stream_object(monkeypatch, kind, n):
    """Large enough to ask, refused by the library: one question, by the stream's number."""
    def no(*a, **k):
        raise AssertionError("a Stream object for a call that does not need it")

    fake = Library()
    monkeypatch.setattr(S, "lib", lambda: fake)
    monkeypatch.setattr(S, "_current_stream", lambda: 7)
    monkeypatch.setattr(torch.cuda, "current_stream", no)
    monkeypatch.setattr(torch.cuda, "stream", no)
    keys = torch.empty(n, dtype=torch.int32)
    assert S._bulk_work(None, kind, keys, None) is None
    assert S._bulk_work(None, kind, keys, 9) is None
    assert fake.asked == [(kind, n, 7), (kind, n, 9)]
    assert S._bulk_work(None, kind, keys[1:], None) is None  # below the line: not even asked
    assert len(fake.asked) == 2
