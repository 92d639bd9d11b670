"""The current stream's handle, also from a torch without the two functions that give
it without the stream object (CPU, torch.cuda replaced)."""

from types import SimpleNamespace

import pytest

from paper_2411_16680_amd import lib

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",),
                                     ("_cuda_getCurrentRawStream", "_cuda_getDevice")])
def test_current_stream(monkeypatch, missing):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=0x1234))
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 3, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: {3: 0x1234}[d], raising=False)
    for name in missing:
        monkeypatch.delattr(torch._C, name)
    assert lib._stream_handle(None) == 0x1234
    assert lib._stream_handle(SimpleNamespace(cuda_stream=7)) == 7
