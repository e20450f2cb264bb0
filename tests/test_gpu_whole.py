"""A whole product formed batch by batch at its place in one output, and the
bound on the columns' entries that a caller may give the numeric pass."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import assert_matches, budget_for_batches

pytestmark = pytest.mark.gpu

S = None


def setup_module(module):
    global S
    import paper_2010_08526_amd as lib
    S = lib
    assert torch.cuda.is_available()


@pytest.mark.parametrize("layers", [1, 3])
@pytest.mark.parametrize("sorted_output", [False, True])
@pytest.mark.parametrize("nb", [1, 4])
def test_whole_product(layers, sorted_output, nb):
    print(f"case: whole layers={layers} sorted={sorted_output} batches={nb}", flush=True)
    A = synth.rmat(13, 12, 3, dtype=torch.float64)
    Ad = A.to("cuda")
    eng = S.Engine(Ad, Ad, layers, sorted_output=sorted_output)
    if nb > 1:
        eng.budget_bytes = budget_for_batches(S, eng, eng.plan(), nb)
    C, plan = eng.run()
    assert (plan.nbatches > 1) == (nb > 1)
    P = oracle.spgemm(A, A)
    assert int(C.colptr[0]) == 0
    if sorted_output:
        assert np.array_equal(C.rowidx.cpu().numpy(), P.rowidx)
    assert_matches(C, P, torch.float64, "whole")
    keep = (C.colptr.clone(), C.rowidx.clone(), C.values.clone())
    Ad.values.mul_(2)
    C2, _ = eng.run()  # the first result is the caller's own
    assert torch.equal(C.colptr, keep[0]) and torch.equal(C.rowidx, keep[1]) and torch.equal(C.values, keep[2])
    Ad.values.mul_(0.5)
    assert torch.equal(C2.colptr, C.colptr)
    parts = []
    eng.run(lambda c0, c1, Cb: parts.append((Cb.rowidx.clone().sort()[0], int(Cb.nnz))))
    assert sum(p[1] for p in parts) == C.nnz


@pytest.mark.parametrize("shape", [(5, 0, 7), (0, 4, 3), (6, 3, 0)])
@pytest.mark.parametrize("layers", [1, 2])
def test_whole_empty(shape, layers):
    print(f"case: whole empty {shape} {layers}", flush=True)
    m, k, n = shape
    z = lambda r, c: S.CSC(r, c, torch.zeros(c + 1, dtype=torch.int64, device="cuda"),  # noqa: E731
                           torch.zeros(0, dtype=torch.int32, device="cuda"), torch.zeros(0, device="cuda"))
    for srt in (False, True):
        C = S.spgemm(z(m, k), z(k, n), layers=layers, sorted_output=srt)
        assert C.colptr.tolist() == [0] * (n + 1) and C.nnz == 0 and C.values.dtype == torch.float32


@pytest.mark.parametrize("limit", [32, 128, 256, 257, 512, 1024, 1025, 2048, 5120])
@pytest.mark.parametrize("sorted_output", [False, True])
def test_bound_on_column_entries(limit, sorted_output):
    """Columns up to the bound are formed; one entry more is reported."""
    print(f"case: bound {limit} sorted={sorted_output}", flush=True)
    m = 9000
    rng = np.random.default_rng(limit)
    I = synth.CSC(m, m, torch.arange(m + 1), torch.arange(m, dtype=torch.int32), torch.ones(m, dtype=torch.float64))
    cols = [np.sort(rng.choice(m, n, replace=False)) for n in (limit, 1, limit - 1)]
    cp = np.concatenate([[0], np.cumsum([c.size for c in cols])]).astype(np.int64)
    B = synth.CSC(m, 3, torch.from_numpy(cp), torch.from_numpy(np.concatenate(cols).astype(np.int32)),
                  torch.from_numpy(rng.standard_normal(int(cp[-1]))))
    A, Bd = I.to("cuda"), B.to("cuda")
    eng = S.Engine(A, Bd)
    plan = eng.plan()
    ws = S.alloc_workspace(S.workspace_size(S.OP_NUMERIC, A, Bd, 0, 3))
    ri = torch.empty(int(cp[-1]), dtype=torch.int32, device="cuda")
    v = torch.empty(int(cp[-1]), dtype=torch.float64, device="cuda")
    t = (torch.empty_like(ri), torch.empty_like(v))
    for bound in (limit, limit - 1):
        if sorted_output:
            S.numeric_sorted(A, Bd, 0, 3, plan.flops, Bd.colptr, ri, v, *t, ws, esc_cf=0.0, max_len=bound)
        else:
            S.numeric(A, Bd, 0, 3, 0, 1, plan.flops, Bd.colptr, ri, v, ws, max_len=bound)
        if bound == limit:
            S.check_many([ws])
            C = S.CSC(m, 3, Bd.colptr, ri, v)
            assert_matches(C, oracle.spgemm(I, B), torch.float64, "bound")
        else:
            with pytest.raises(S.SpgemmError, match="device code 4"):
                S.check_many([eng.ws_sym, ws])
            S.check_many([ws])  # reported once


@pytest.mark.parametrize("layers", [1, 3])
@pytest.mark.parametrize("sorted_output", [False, True])
def test_plan_from_device_sums(layers, sorted_output):
    """A product of enough columns to be planned from sums on the device: the
    same plan as the planner's, at the smallest budget that holds it whole and
    one byte below; counts read back later are those of their own product."""
    print(f"case: device sums layers={layers} sorted={sorted_output}", flush=True)
    A = synth.erdos_renyi(40000, 40000, 3, 5, torch.float32)
    B = synth.erdos_renyi(40000, 40000, 5, 6, torch.float32)
    eng = S.Engine(A.to("cuda"), B.to("cuda"), layers, sorted_output=sorted_output)
    plan = eng.plan()
    assert isinstance(plan.counts, torch.Tensor)  # not read back yet
    first = eng.plan()
    eng.B.rowidx[:1000] = eng.B.rowidx[0]  # another product in the same engine
    eng.plan()
    want = oracle.count(A, B)
    assert np.array_equal(plan.nnz_host[-1], want) and np.array_equal(first.nnz_host, plan.nnz_host)
    assert plan.longest == want.max() and plan.bounds == [0, 40000]
    assert np.array_equal(plan.batch_nnz, plan.nnz_host.sum(1)[None])
    eng = S.Engine(A.to("cuda"), B.to("cuda"), layers, sorted_output=sorted_output)
    u = plan.nnz_host.sum(1)
    held = int(u[-1]) * (2 if sorted_output else 1) + (int(u[:-1].sum()) if layers > 1 else 0)
    need = 8 * held + 8 * (layers + 1 if layers > 1 else 1) * 40000
    for extra, nb in ((0, 1), (-1, 2)):
        eng.budget_bytes = eng.input_bytes + eng.reserve_bytes + need + extra
        assert eng.plan().nbatches == nb
    eng.budget_bytes = eng.input_bytes + eng.reserve_bytes
    with pytest.raises(S.SpgemmError):
        eng.plan()


@pytest.mark.parametrize("n", [40, 9000])
def test_layers_below_the_merged_length(n):
    """Columns of more than 5120 rows of which no layer forms more: every
    count's longest column is planned with (from the host and from sums on the
    device), and the product is the oracle's."""
    print(f"case: layers below the merged length {n}", flush=True)
    m, k, L = 20000, 800, 4
    A = synth.erdos_renyi(m, k, 40, 5, torch.float64)
    few = synth.erdos_renyi(k, n - 8, 2, 6, torch.float64)
    many = synth.erdos_renyi(k, 8, 300, 7, torch.float64)
    B = synth.CSC(k, n, torch.cat([few.colptr, many.colptr[1:] + few.nnz]), torch.cat([few.rowidx, many.rowidx]),
                  torch.cat([few.values, many.values]))
    eng = S.Engine(A.to("cuda"), B.to("cuda"), L)
    C, plan = eng.run()
    P = oracle.spgemm(A, B)
    assert (plan.nnz_host.size >= 32768) == (n == 9000)
    assert np.array_equal(plan.row_longest, plan.nnz_host.max(axis=1))
    assert plan.row_longest[:L].max() <= 5120 < plan.longest == np.diff(P.colptr).max()
    assert_matches(C, P, torch.float64, "layers")
