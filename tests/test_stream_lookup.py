"""The current stream is looked up by names that torch does not promise: a torch without them is asked the public way."""
import types

import pytest
import torch

from paper_2305_12213_amd import binding


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_torch_without_the_private_names(monkeypatch, missing):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 56, raising=False)
    assert binding._stream(None) == 56
    monkeypatch.delattr(torch._C, missing)
    assert binding._stream(None) == 1234
    assert binding._stream(7) == 7
