"""Plans that a program makes, changes or saves itself (no GPU)."""
from __future__ import annotations

import copy
import dataclasses
import pickle

import numpy as np
import torch

import paper_2010_08526_amd as S

FIELDS = ["flops", "nnz", "nnz_host", "bounds", "batch_nnz", "n_layers", "budget_bytes", "input_bytes",
          "reserve_bytes"]


def _values():
    counts = np.arange(1, 7, dtype=np.int64).reshape(1, 6)
    return [torch.ones(6, dtype=torch.int64), torch.from_numpy(counts), counts, [0, 4, 6], np.array([[10], [11]]), 1,
            1000, 10, 20]


def test_plan_is_made_from_its_fields():
    """By position and by name, with the fields a plan has always had."""
    v = _values()
    for p in (S.Plan(*v), S.Plan(**dict(zip(FIELDS, v)))):
        assert [f.name for f in dataclasses.fields(p)][:9] == FIELDS
        assert p.nnz_host is v[2] and p.bounds == [0, 4, 6] and p.nbatches == 2 and p.total_flops == 6
    q = dataclasses.replace(p, bounds=[0, 6], batch_nnz=np.array([[21]]))
    assert q.nnz_host is v[2] and q.nbatches == 1
    p.nnz_host = v[2] * 2
    assert np.array_equal(p.nnz_host, v[2] * 2)


def test_saved_plans():
    """A plan survives copying and pickling, and one saved without the length
    of its longest column loads."""
    v = _values()
    for p in (S.Plan(*v), S.Plan(*v, longest=6)):
        for q in (pickle.loads(pickle.dumps(p)), copy.copy(p), copy.deepcopy(p)):
            assert np.array_equal(q.nnz_host, v[2]) and q.longest == p.longest and q.bounds == p.bounds
    old = S.Plan.__new__(S.Plan)
    old.__dict__.update(zip(FIELDS, v))  # as a saved plan is loaded
    assert np.array_equal(old.nnz_host, v[2]) and old.longest is None


def test_plan_without_a_bound(monkeypatch):
    """A plan that does not say how long columns are puts no bound on them."""
    bounds = []
    monkeypatch.setattr(S, "numeric", lambda *a: bounds.append(a[-1]))
    eng = object.__new__(S.Engine)
    eng.A = eng.B = S.CSC(4, 6, None, torch.zeros(0), None)
    eng.L, eng.sorted_output, eng.semiring, eng.flops, eng.ws_num = 1, False, 0, torch.zeros(6), None
    for longest, want in ((None, S.NO_BOUND), (6, 6)):
        plan = S.Plan(*_values(), longest=longest)
        eng._form(plan, 0, None, 10, [], (None, None), (None, None))
        assert bounds.pop() == want


def test_layers_have_bounds_of_their_own(monkeypatch):
    """A layer's product is bounded by its own longest column, not by C's."""
    bounds = []
    monkeypatch.setattr(S, "numeric", lambda *a: bounds.append(a[-1]))
    monkeypatch.setattr(S, "merge", lambda *a: None)
    eng = object.__new__(S.Engine)
    eng.A = eng.B = S.CSC(4, 6, None, torch.zeros(0), None)
    eng.L, eng.sorted_output, eng.semiring, eng.flops = 2, False, 0, torch.zeros(6)
    eng.ws_num = eng.ws_mrg = None
    parts = [S.CSC(4, 6, None, None, None)] * 2
    for more, want in (({}, [S.NO_BOUND] * 2), ({"longest": 6}, [6, 6]),
                       ({"longest": 6, "row_longest": np.array([2, 4, 6])}, [2, 4])):
        eng._form(S.Plan(*_values(), **more), 0, None, 10, parts, (None, None), (None, None))
        assert bounds == want
        bounds.clear()
