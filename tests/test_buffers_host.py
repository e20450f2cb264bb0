"""What an engine holds between products, checked without a GPU."""
from __future__ import annotations

import types

import numpy as np
import pytest
import torch

import paper_2010_08526_amd as S


def _engine(monkeypatch, layers, sorted_output):
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=0))
    for name in ("colptr", "numeric", "numeric_sorted", "merge"):
        monkeypatch.setattr(S, name, lambda *a: None)
    monkeypatch.setattr(S._lib, "spgemm_sort_columns", lambda *a: 0)
    eng = object.__new__(S.Engine)
    eng.A = eng.B = S.CSC(50, 6, None, torch.zeros(0), None)
    eng.L, eng.vbytes, eng.vdtype, eng.sorted_output = layers, 8, torch.float64, sorted_output
    eng.semiring, eng.esc_cf, eng.device, eng._bufs = 0, 2.0, "cpu", {}
    eng.ws_scan = eng.ws_num = eng.ws_mrg = eng.ws_sort = torch.zeros(16)
    eng.flops = torch.zeros(6)
    eng.nnz = torch.ones((layers + 1 if layers > 1 else 1, 6), dtype=torch.int64)
    return eng


def _plan(layers, part, out):
    """Two batches of 4 and 2 columns; `part` entries a layer and `out` merged in the first."""
    rows = [[part] * layers + [out], [1] * layers + [1]] if layers > 1 else [[out], [1]]
    return types.SimpleNamespace(batch_nnz=np.array(rows), nbatches=2, bounds=[0, 4, 6], longest=None, row_longest=None)


def _held(eng):
    return {k: (t.data_ptr(), t.numel()) for k, t in eng._bufs.items()}


@pytest.mark.parametrize("layers", [1, 3])
@pytest.mark.parametrize("sorted_output", [False, True])
def test_one_set_of_buffers(monkeypatch, layers, sorted_output):
    """Products returned whole and batch by batch share their staging: an
    engine used both ways holds no more than it needs for either."""
    eng = _engine(monkeypatch, layers, sorted_output)
    plan = _plan(layers, 30, 40)
    C = eng.run_batch(plan, 0)
    assert C.ncols == 4 and C.nnz == 40 and C.colptr.numel() == 5
    assert eng.run_batch(plan, 1).nnz == 1
    before = _held(eng)
    assert eng._whole(plan).nnz == 41
    for name in set(before) - {"dcp"}:  # (pointers of all columns)
        assert _held(eng)[name] == before[name]
    sizes = {k: n for k, (_, n) in _held(eng).items()}
    want = {"ccp": 5, "cri": 40, "cv": 40}
    if sorted_output:
        want.update(sri=40, sv=40)
    if layers > 1:
        want.update(dri=90, dv=90, dcp=3 * 6 + 1)
        sizes.pop("wcp")
    assert sizes == want
    eng.release_buffers()
    eng._whole(plan)
    names = ({"cri", "cv"} if sorted_output else set()) | ({"dri", "dv", "dcp", "wcp"} if layers > 1 else set())
    assert set(_held(eng)) == names


def test_buffers_grow_to_the_largest(monkeypatch):
    """Plans of opposite shapes in turn: after one of each, nothing is
    allocated any more."""
    eng = _engine(monkeypatch, 3, True)
    plans = [_plan(3, 30, 5), _plan(3, 2, 70)]
    for form in (eng._whole, lambda p: eng.run_batch(p, 0)):
        for p in plans:
            form(p)
        before = _held(eng)
        assert before["dri"][1] == 90 and before["cri"][1] == 70
        for p in plans * 2:
            form(p)
            assert _held(eng) == before
