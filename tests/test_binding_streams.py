"""The binding's stream handle and clearing, with and without the torch names
that make them cheap."""
import pytest

torch = pytest.importorskip("torch")
from paper_2607_24062_amd import acrl  # noqa: E402


class _Stream:
    cuda_stream = 1234


@pytest.mark.parametrize("raw", [None, lambda index: 77])
def test_raw_stream(monkeypatch, raw):
    monkeypatch.setattr(acrl, "_current_raw", raw)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: _Stream())
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    want = 1234 if raw is None else 77
    assert acrl._raw_stream() == want
    assert acrl._raw_stream(None, torch.device("cuda:0")) == want
    other = type("S", (), {"cuda_stream": 9})()
    assert acrl._raw_stream(other) == 9 and acrl._raw_stream(other, torch.device("cuda:0")) == 9


def test_host_tensors_have_no_stream():
    with pytest.raises((ValueError, RuntimeError, AssertionError)):
        acrl._raw_stream(None, torch.device("cpu"))


@pytest.mark.parametrize("all_at_once", [None, torch._foreach_zero_])
def test_zero(monkeypatch, all_at_once):
    monkeypatch.setattr(acrl, "_zero_all", all_at_once)
    ts = [torch.ones(5), torch.ones(7)]
    acrl._zero(ts)
    assert all(not bool(t.any()) for t in ts)
