"""The binding's current stream without torch's private shortcut to its handle, and with it."""
from types import SimpleNamespace

from paper_2406_11674_amd import binding


def _torch(**private):
    cuda = SimpleNamespace(current_device=lambda: 3, current_stream=lambda: SimpleNamespace(cuda_stream=0x77))
    return SimpleNamespace(_C=SimpleNamespace(**private), cuda=cuda)


def test_without_the_private_name(monkeypatch):
    monkeypatch.setattr(binding, "_torch", lambda: _torch())
    assert binding._stream_handle(None) == 0x77
    assert binding._stream_handle(SimpleNamespace(cuda_stream=5)) == 5


def test_with_it(monkeypatch):
    monkeypatch.setattr(binding, "_torch", lambda: _torch(_cuda_getCurrentRawStream=lambda device: 100 + device))
    assert binding._stream_handle(None) == 103
