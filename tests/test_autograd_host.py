"""What autograd sees of the binding, checked without a GPU."""
from __future__ import annotations

import types

import pytest
import torch

import paper_2010_08526_amd as S


def test_kept_values_are_no_part_of_a_graph(monkeypatch):
    """A Backward made, and refreshed, with values that require gradients
    records nothing: its copy of them has no history that could grow."""
    monkeypatch.setattr(S, "alloc_workspace", lambda *a: torch.zeros(256, dtype=torch.uint8))
    v = torch.ones(4, requires_grad=True)
    M = S.CSC(4, 4, torch.arange(5), torch.arange(4, dtype=torch.int32), v)
    bw = S.Backward(M, M, M)
    assert bw.ws_f is not None
    for k in range(3):
        assert not bw._b.requires_grad and bw._b.grad_fn is None
        assert torch.equal(bw._b, M.values)
        M.values = v * (k + 2)
        bw.refresh_values(M)


def test_undefined_gradient_counts_as_zero():
    """A consumer of C's values that has no gradient for them: dA and dB are
    zeros (not missing)."""
    a, b = torch.ones(5), torch.ones(7)
    dA, dB, *rest = S.SpGEMMFn.backward(types.SimpleNamespace(saved_tensors=(a, b)), None, None, None)
    assert torch.equal(dA, torch.zeros(5)) and torch.equal(dB, torch.zeros(7)) and rest == [None] * 4


@pytest.mark.parametrize("row, nnz_c, hub", [(4096, 4096, False), (4097, 4097, True), (4097, 128 * 4097 - 1, True),
                                             (4097, 128 * 4097, False), (10**7, 10**9, True), (0, 0, False)])
def test_rule_of_the_fused_gradients(row, nnz_c, hub):
    assert S._hub_row(row, row, nnz_c) == hub and S._hub_row(row, nnz_c, 0) == hub
