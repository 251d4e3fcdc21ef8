"""The stream a call without a stream argument runs on: torch's current one, also
with a torch that has no raw-handle function, and the device initialised as torch's
own call would (CPU; the device functions are replaced)."""

import types

import pytest

torch = pytest.importorskip("torch")

from paper_2605_04864_amd import _lib as L  # noqa: E402


def test_raw_handle_of_the_current_device(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 1000 + dev, raising=False)
    assert L.stream_handle() == 1003


def test_public_stream_without_raw_handles(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=77))
    assert L.stream_handle() == 77


def test_given_stream():
    assert L.stream_handle(types.SimpleNamespace(cuda_stream=5)) == 5


@pytest.mark.gpu
def test_current_stream_on_the_device():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    s = torch.cuda.Stream()
    assert L.stream_handle() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(s):
        assert L.stream_handle() == s.cuda_stream
