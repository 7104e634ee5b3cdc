"""The binding's default stream (CPU, with torch's stream calls replaced): the
handle asked for directly where torch has the call, the public one where not."""
from types import SimpleNamespace

import pytest

from paper_2609_36760_amd import _binding as mb


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",),
                                     ("_cuda_getCurrentRawStream", "_cuda_getDevice")])
def test_default_stream(monkeypatch, missing):
    import torch
    direct = {"_cuda_getCurrentRawStream": lambda device: 100 + device, "_cuda_getDevice": lambda: 3}
    for name, call in direct.items():
        if name in missing:
            monkeypatch.delattr(torch._C, name, raising=False)
        else:
            monkeypatch.setattr(torch._C, name, call, raising=False)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=7))
    monkeypatch.setattr(mb, "_current_stream", None, raising=False)
    assert [mb._stream(None) for _ in range(2)] == ([7, 7] if missing else [103, 103])
    assert mb._stream(5) == 5 and mb._stream(SimpleNamespace(cuda_stream=9)) == 9
