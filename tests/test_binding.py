"""CPU-only checks of the binding itself."""
import importlib.util

import pytest
import torch

from paper_2406_09904_amd import binding


@pytest.mark.parametrize("missing", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_stream_handle_without_torchs_private_names(monkeypatch, missing):
    """A torch without one of them: the handle comes from torch.cuda.current_stream()."""
    class Stream:
        cuda_stream = 0x1234

    monkeypatch.delattr(torch._C, missing, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: Stream if device == 3 else None)
    spec = importlib.util.spec_from_file_location("binding_without_" + missing, binding.__file__)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    assert module._stream() == 0x1234
    assert module._raw_stream(module._device()) == 0x1234
