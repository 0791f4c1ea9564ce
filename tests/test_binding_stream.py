"""The binding launches on torch's current stream, by the private query for its handle or, in a
torch that does not have it, by the public one."""
import types

import torch

from paper_2510_07729_amd import sop


def test_stream_handle_with_and_without_the_private_query(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream",
                        lambda *a: types.SimpleNamespace(cuda_stream=11))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 100 + d, raising=False)
    assert sop._stream() == 103
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert sop._stream() == 11
