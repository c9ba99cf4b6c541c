"""The current stream's handle, with and without torch's private short cut."""
import importlib.util
import types

import pytest
import torch

from paper_1809_11134_amd import qe


@pytest.mark.parametrize("short_cut", [True, False])
def test_current_stream_handle(monkeypatch, short_cut):
    handle = 0x7F12_3456_789A                          # (more than 32 bits)
    if short_cut:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: handle + dev, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=handle))
    spec = importlib.util.spec_from_file_location("qe_without_short_cut", qe.__file__)
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    assert module._stream(None) == handle
    assert module._stream(types.SimpleNamespace(cuda_stream=5)) == 5
