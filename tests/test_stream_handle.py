"""The stream that a call without one runs on, with no GPU: torch's current one, also where torch has no function for the bare handle."""
import types

import torch

from paper_2410_11415_amd import Circuit


def test_without_the_bare_handle(monkeypatch):
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=4711))
    assert Circuit._stream(None) == 4711


def test_a_given_stream():
    assert Circuit._stream(types.SimpleNamespace(cuda_stream=13)) == 13
