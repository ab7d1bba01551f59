"""The stream handle of the Python calls: the raw-handle function that a PyTorch
build may not have is a shortcut for the public current_stream, not a need."""
import importlib.util
import types

import torch

import paper_2504_15508_amd.plan as plan


def test_public_stream_without_the_raw_handle(monkeypatch):
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    spec = importlib.util.spec_from_file_location("paper_2504_15508_amd._plan_without_raw", plan.__file__)
    copy = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(copy)
    asked = []
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda d: asked.append(d) or types.SimpleNamespace(cuda_stream=0x7F00_1234_5678))
    dev = torch.device("cuda", 1)
    assert copy._stream(dev) == 0x7F00_1234_5678 and asked == [dev]
