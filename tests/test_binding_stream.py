"""The stream handle the binding passes, on the CPU."""
import types

import torch

from paper_2604_16590_amd import _binding as b


def test_stream_without_torchs_private_call(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(b, "_raw_stream", None, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device: types.SimpleNamespace(cuda_stream=1234))
    assert b._stream(torch.device("cuda:0")) == 1234
    assert b._stream(torch.device("cuda")) == 1234
