"""The stream handle the binding passes to the library where PyTorch does not have the short route to it."""
import torch

import paper_1901_09971_amd.api as api


def test_stream_without_the_private_names(monkeypatch):
    class Stream:
        def __init__(self, device):
            self.cuda_stream = 4096 + device

    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream(3 if device is None else device))
    monkeypatch.setattr(api, "_raw_stream", api._raw_stream_getter())
    assert api._stream() == 4096 + 3
