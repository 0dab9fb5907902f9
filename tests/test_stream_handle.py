"""The binding's stream handle where PyTorch has no raw-stream call."""
import types

import torch

from paper_1602_08604_amd import lre as L


def test_public_api_serves(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    monkeypatch.setattr(L, "_raw_stream", None, raising=False)
    asked = []
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda device: asked.append(device) or types.SimpleNamespace(cuda_stream=4711))
    device = torch.device("cuda", 0)
    assert L._stream(device) == 4711 and asked == [device]
