"""The current stream's handle with and without torch's private shortcut."""
import types

import torch

import paper_2310_03121_amd as nnp


def test_public_way_without_the_shortcut(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda: types.SimpleNamespace(cuda_stream=1234))
    assert nnp._stream() == 1234


def test_shortcut(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 100 + device,
                        raising=False)
    assert nnp._stream() == 103
