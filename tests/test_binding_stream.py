"""The handle of the current stream, with and without torch's short way to it."""
import types

from paper_2605_23163_amd import binding


def fake_torch(**c):
    stream = types.SimpleNamespace(cuda_stream=77)
    return types.SimpleNamespace(_C=types.SimpleNamespace(**c),
                                 cuda=types.SimpleNamespace(current_stream=lambda: stream, current_device=lambda: 3))


def test_stream_handle(monkeypatch):
    monkeypatch.setattr(binding, "torch", fake_torch(_cuda_getCurrentRawStream=lambda d: 70 + d))
    assert binding._stream_ptr(None) == 73
    monkeypatch.setattr(binding, "torch", fake_torch())
    assert binding._stream_ptr(None) == 77
    assert binding._stream_ptr(types.SimpleNamespace(cuda_stream=5)) == 5
