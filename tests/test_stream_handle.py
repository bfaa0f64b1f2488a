"""The stream handle the binding passes on: the given one, or that of torch's
current stream on the current device, with and without torch's raw accessors
(stand-ins for torch.cuda; no GPU)."""
import types

import pytest

from paper_2606_11440_amd import _lib


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",)])
def test_current_stream_handle(monkeypatch, missing):
    import torch
    at = {"device": 0}
    raw = {"_cuda_getCurrentRawStream": lambda d: 100 + d, "_cuda_getDevice": lambda: at["device"]}
    for name, f in raw.items():
        if name in missing:
            monkeypatch.delattr(torch._C, name, raising=False)
        else:
            monkeypatch.setattr(torch._C, name, f, raising=False)
    monkeypatch.setattr(torch.cuda, "init", lambda: None)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: at["device"])
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d: types.SimpleNamespace(cuda_stream=100 + d))
    monkeypatch.setattr(_lib, "_current", None)
    for at["device"] in (0, 3):
        assert _lib._stream(None) == 100 + at["device"]
    assert _lib._stream(7) == 7
