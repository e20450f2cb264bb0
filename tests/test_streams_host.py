"""Streams that the binding gives to torch's own work, checked without a GPU:
torch's stream calls are replaced by stand-ins that record what is asked for."""
from __future__ import annotations

import types

import pytest
import torch

import paper_2010_08526_amd as S


class FakeCuda:
    """Stand-ins for torch.cuda's streams; `entered` lists the handles whose
    context was entered (an external stream of handle 0 is another stream)."""

    def __init__(self, monkeypatch, current):
        self.entered = []
        stream = lambda h: types.SimpleNamespace(cuda_stream=h)  # noqa: E731
        monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: stream(current))
        monkeypatch.setattr(torch.cuda, "default_stream", lambda *a: stream(0))
        monkeypatch.setattr(torch.cuda, "ExternalStream", lambda h: stream(h if h else "another stream"))
        monkeypatch.setattr(torch.cuda, "stream", self.enter)

    def enter(self, s):
        self.entered.append(s.cuda_stream)
        return types.SimpleNamespace(__enter__=lambda: s, __exit__=lambda *a: None)


@pytest.mark.parametrize("current", [0, 4096])
@pytest.mark.parametrize("handle", [None, 0, 4096, 8192])
def test_context_of_a_handle(monkeypatch, current, handle):
    """The context of a handle is that stream, for handle 0 the default one."""
    fake = FakeCuda(monkeypatch, current)
    S._on_stream(handle)
    used = fake.entered[0] if fake.entered else current
    assert used == (current if handle is None else handle)
