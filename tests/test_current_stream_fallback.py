"""The binding asks torch for the current stream's handle by functions that are not public where torch has them, and by the
public ones where it has not (CPU only)."""
import types

import pytest
import torch

from paper_2506_12024_amd import binding


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_a_torch_without_the_raw_functions(monkeypatch, missing):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 40 + device, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 2, raising=False)
    assert binding._stream(None) == 42
    monkeypatch.delattr(torch._C, missing)
    assert binding._stream(None) == 77
