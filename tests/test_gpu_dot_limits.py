"""GPU parity of the masked products at the edges of their classes: table
sizes of Y(:,j) (full and half tables), entries of M(:,j) shared among one to
sixteen waves, and columns of X from empty to longer than a wave's walk."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

S = None
YLEN = [0, 1, 32, 33, 128, 129, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 5120, 5121]
MLEN = [0, 1, 3, 4, 5, 63, 64, 65, 257, 1100]
XLEN = [0, 1, 2, 3, 5, 31, 62, 63, 64, 65, 130, 300]


def setup_module(module):
    global S
    import paper_2010_08526_amd as lib
    S = lib
    assert torch.cuda.is_available()


def _csc(m, cols, rng, dtype):
    cp = np.concatenate([[0], np.cumsum([c.size for c in cols])]).astype(np.int64)
    ri = np.concatenate(cols).astype(np.int32)
    return synth.CSC(m, len(cols), torch.from_numpy(cp), torch.from_numpy(ri),
                     torch.from_numpy(rng.integers(1, 9, ri.size)).to(dtype))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("mix", ["mixed", "short", "long"])
def test_masked_product_limits(dtype, mix):
    """Values are small integers, so every dot product is exact."""
    print(f"case: masked product limits {mix} {dtype}", flush=True)
    rng = np.random.default_rng(len(mix))
    m = 6000
    xl = {"mixed": XLEN, "short": [0, 1, 2, 3], "long": [63, 64, 130, 300]}[mix]
    X = _csc(m, [rng.choice(m, xl[i % len(xl)], replace=False) for i in range(1200)], rng, dtype)
    Y = _csc(m, [rng.choice(m, n, replace=False) for n in YLEN for _ in MLEN], rng, dtype)
    M = _csc(X.ncols, [rng.choice(X.ncols, n, replace=False) for _ in YLEN for n in MLEN], rng, dtype)
    got = S.masked_xty(X.to("cuda"), Y.to("cuda"), M.to("cuda"))
    assert np.array_equal(got.double().cpu().numpy(), oracle.masked_xty(X, Y, M))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("n", [768, 769, 3072, 3073])
def test_half_tables_by_columns(n, dtype):
    """As many columns as take full tables only, and one more than that for
    either of the bins with half tables: products, masked products and both
    gradients of columns at the tables' limits; exact."""
    print(f"case: half tables {n} {dtype}", flush=True)
    rng = np.random.default_rng(n)
    m = 2100
    lens = [128, 129, 256, 257, 512, 513, 1024, 1025, 2048]
    one = _csc(m, [np.array([i]) for i in range(m)], rng, dtype)  # columns of one entry
    B = _csc(m, [rng.permutation(m)[:lens[j % len(lens)]] for j in range(n)], rng, dtype)
    A, Bd = one.to("cuda"), B.to("cuda")
    C = S.spgemm(A, Bd, sorted_output=True)
    P = oracle.spgemm(one, B)
    assert np.array_equal(C.colptr.cpu().numpy(), P.colptr) and np.array_equal(C.rowidx.cpu().numpy(), P.rowidx)
    assert np.array_equal(C.values.double().cpu().numpy(), P.values)
    H = S.spgemm(A, Bd, layers=3)  # merged
    order = np.lexsort((H.rowidx.cpu().numpy(), np.repeat(np.arange(n), np.diff(P.colptr))))
    assert np.array_equal(H.values.double().cpu().numpy()[order], P.values)
    M = _csc(m, [rng.permutation(m)[:5 + j % 3] for j in range(n)], rng, dtype)
    got = S.masked_xty(A, C, M.to("cuda"))
    assert np.array_equal(got.double().cpu().numpy(), oracle.masked_xty(one, P, M))
    bw = S.Backward(A, Bd, C)
    dA, dB = bw(C.values)
    bw.check()
    assert bw.ws_f is not None
    G = oracle.Mat(m, n, P.colptr, P.rowidx, P.values)
    assert np.array_equal(dA.double().cpu().numpy(), oracle.grad_a(one, B, G).astype(np.float32 if dtype == torch.float32 else np.float64))
    assert np.array_equal(dB.double().cpu().numpy(), oracle.grad_b(one, B, G))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_gradient_limits(dtype):
    """Both gradients of products whose columns hold 1 to 5120 rows, the
    entries of B ranging from one per column to several per wave; exact."""
    print(f"case: gradient limits {dtype}", flush=True)
    rng = np.random.default_rng(5)
    m = 6000
    lens = [1, 2, 16, 63, 64, 65, 128]
    A = _csc(m, [np.arange(s, s + n) for n in lens for s in rng.integers(0, m - 200, 60)], rng, dtype)
    cols = [rng.choice(A.ncols, n, replace=False) for n in (1, 2, 3, 5, 8, 13, 21, 34, 64, 65, 130) for _ in range(4)]
    B = _csc(A.ncols, cols, rng, dtype)
    Ad, Bd = A.to("cuda"), B.to("cuda")
    C = S.spgemm(Ad, Bd)
    assert int((C.colptr[1:] - C.colptr[:-1]).max()) > 2048
    dC = torch.from_numpy(rng.integers(1, 5, C.nnz)).to(dtype).cuda()
    bw = S.Backward(Ad, Bd, C)
    dA, dB = bw(dC)
    bw.check()
    G = oracle.Mat(C.nrows, C.ncols, C.colptr.cpu().numpy(), C.rowidx.cpu().numpy(), dC.double().cpu().numpy())
    assert np.array_equal(dA.double().cpu().numpy(), oracle.grad_a(A, B, G))
    assert np.array_equal(dB.double().cpu().numpy(), oracle.grad_b(A, B, G))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_backward_forms_agree(dtype, monkeypatch):
    """Gradients in one traversal and by transposed patterns: the same exact
    values (small integers) for the values B had at construction or at the last
    refresh; transposed patterns of the first form made on request; a dC of
    another type is refused by both."""
    print(f"case: backward forms {dtype}", flush=True)
    rng = np.random.default_rng(8)
    A = _csc(500, [rng.choice(500, n, replace=False) for n in rng.integers(0, 90, 300)], rng, dtype).to("cuda")
    B = _csc(300, [rng.choice(300, n, replace=False) for n in rng.integers(0, 70, 200)], rng, dtype).to("cuda")
    C = S.spgemm(A, B)
    dC = torch.from_numpy(rng.integers(1, 5, C.nnz)).to(dtype).cuda()
    fused = S.Backward(A, B, C)
    monkeypatch.setattr(S, "FUSED_COL_MAX", 0)
    trans = S.Backward(A, B, C)
    assert fused.ws_f is not None and trans.ws_f is None

    def same():
        for x, y in zip(fused(dC), trans(dC)):
            assert x.dtype == dtype and torch.equal(x, y)
        fused.check()
        trans.check()

    same()
    B.values.mul_(3)  # not seen before a refresh
    same()
    B2 = S.CSC(B.nrows, B.ncols, B.colptr, B.rowidx, B.values + 1)
    fused.refresh_values(B2)
    trans.refresh_values(B2)
    same()
    BT = fused.BT
    assert torch.equal(BT.colptr, trans.BT.colptr)
    fused.refresh_values(B)
    assert torch.equal(fused.BT.values, B.values[fused.permB])
    other = torch.float64 if dtype == torch.float32 else torch.float32
    for bw in (fused, trans):
        with pytest.raises(S.SpgemmError):
            bw(dC.to(other))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_gradient_over_an_input(dtype):
    """dA written over A's own values: the terms have read them by then."""
    print(f"case: gradient over an input {dtype}", flush=True)
    import ctypes
    rng = np.random.default_rng(2)
    A = _csc(400, [rng.choice(400, n, replace=False) for n in rng.integers(0, 80, 200)], rng, dtype).to("cuda")
    B = _csc(200, [rng.choice(200, n, replace=False) for n in rng.integers(0, 60, 150)], rng, dtype).to("cuda")
    C = S.spgemm(A, B)
    dC = torch.from_numpy(rng.integers(1, 5, C.nnz)).to(dtype).cuda()
    wA, wB = S.Backward(A, B, C)(dC)
    ws = S.alloc_workspace(S.workspace_size(S.OP_BATCHED_BACKWARD, A, B, 0, C.ncols))
    dB = torch.empty_like(B.values)
    cd = S.desc(S.CSC(C.nrows, C.ncols, C.colptr, C.rowidx, None), S.F32)
    S._check(S._lib.spgemm_batched_backward(ctypes.byref(S.desc(A)), ctypes.byref(S.desc(B)), ctypes.byref(cd),
                                            S._ptr(dC), S._ptr(A.values), S._ptr(dB), S._ptr(ws), ws.numel(),
                                            S._stream(None)), "spgemm_batched_backward")
    S.check_ws(ws)
    assert torch.equal(A.values, wA) and torch.equal(dB, wB)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("shape", [(6, 3, 0), (5, 0, 7), (0, 4, 3)])
def test_gradients_of_empty_products(shape, dtype):
    """No columns, no inner dimension, no rows: gradients of zeros."""
    print(f"case: empty gradients {shape} {dtype}", flush=True)
    m, k, n = shape
    A = synth.erdos_renyi(m, k, min(m, 2), 3, dtype).to("cuda")
    B = synth.erdos_renyi(k, n, min(k, 2), 4, dtype).to("cuda")
    C = S.spgemm(A, B)
    assert C.nnz == 0
    bw = S.Backward(A, B, C)
    dA, dB = bw(C.values)
    bw.check()
    assert torch.equal(dA, torch.zeros_like(A.values)) and torch.equal(dB, torch.zeros_like(B.values))
    a, b = A.values.clone().requires_grad_(True), B.values.clone().requires_grad_(True)
    S.SpGEMMFn.apply(a, b, A, B)[0].sum().backward()
    assert torch.equal(a.grad, torch.zeros_like(a)) and torch.equal(b.grad, torch.zeros_like(b))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("row", [4096, 4097])
def test_gradients_with_a_long_row(row, dtype):
    """A row of B in 4096 columns (one traversal) and in one more (transposed
    patterns), of few other entries; exact."""
    print(f"case: gradients with a long row {row} {dtype}", flush=True)
    rng = np.random.default_rng(row)
    n = 6000
    A = _csc(300, [rng.choice(300, 8, replace=False) for _ in range(50)], rng, dtype)
    B = _csc(50, [np.array([7, 20]) if j < row else np.array([j % 7]) for j in rng.permutation(n)], rng, dtype)
    Ad, Bd = A.to("cuda"), B.to("cuda")
    C = S.spgemm(Ad, Bd)
    dC = torch.from_numpy(rng.integers(1, 5, C.nnz)).to(dtype).cuda()
    bw = S.Backward(Ad, Bd, C)
    assert S._longest_row(Bd) == row and (bw.ws_f is None) == (row > 4096)
    G = oracle.Mat(C.nrows, C.ncols, C.colptr.cpu().numpy(), C.rowidx.cpu().numpy(), dC.double().cpu().numpy())
    gA, gB = oracle.grad_a(A, B, G), oracle.grad_b(A, B, G)
    for k in (1, 3):
        dA, dB = bw(dC)
        bw.check()
        assert np.array_equal(dA.double().cpu().numpy(), k * gA)
        assert np.array_equal(dB.double().cpu().numpy(), gB)
        bw.refresh_values(S.CSC(Bd.nrows, n, Bd.colptr, Bd.rowidx, Bd.values * 3))


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("longest", [5120, 5121])
def test_form_of_the_gradients_at_the_limit(longest, dtype, monkeypatch):
    """C's longest column has as many rows as the largest table takes, or one
    more: one traversal, or transposed patterns, by Backward and by SpGEMMFn;
    exact."""
    print(f"case: form of the gradients {longest} {dtype}", flush=True)
    rng = np.random.default_rng(longest)
    m = 6000
    rows = rng.permutation(m)[:longest]
    A = _csc(m, [rows[i:i + 64] for i in range(0, longest, 64)] + [rng.choice(m, 3, replace=False)], rng, dtype)
    B = _csc(A.ncols, [np.arange(A.ncols - 1), np.array([A.ncols - 1]), np.array([0, A.ncols - 2])], rng, dtype)
    Ad, Bd = A.to("cuda"), B.to("cuda")
    C = S.spgemm(Ad, Bd)
    assert int((C.colptr[1:] - C.colptr[:-1]).max()) == longest
    dC = torch.from_numpy(rng.integers(1, 5, C.nnz)).to(dtype).cuda()
    bw = S.Backward(Ad, Bd, C)
    assert (bw.ws_f is not None) == (longest == 5120)
    dA, dB = bw(dC)
    bw.check()
    G = oracle.Mat(C.nrows, C.ncols, C.colptr.cpu().numpy(), C.rowidx.cpu().numpy(), dC.double().cpu().numpy())
    gA, gB = oracle.grad_a(A, B, G), oracle.grad_b(A, B, G)
    assert np.array_equal(dA.double().cpu().numpy(), gA) and np.array_equal(dB.double().cpu().numpy(), gB)

    formed = []
    monkeypatch.setattr(S, "_fused_backward", lambda *a, f=S._fused_backward: formed.append(1) or f(*a))
    a, b = Ad.values.clone().requires_grad_(True), Bd.values.clone().requires_grad_(True)
    c, cp, ri = S.SpGEMMFn.apply(a, b, Ad, Bd)
    c.backward(torch.ones_like(c))
    assert len(formed) == (longest == 5120)
    G = oracle.Mat(C.nrows, C.ncols, cp.cpu().numpy(), ri.cpu().numpy(), np.ones(C.nnz))
    assert np.array_equal(a.grad.double().cpu().numpy(), oracle.grad_a(A, B, G))
    assert np.array_equal(b.grad.double().cpu().numpy(), oracle.grad_b(A, B, G))


@pytest.mark.parametrize("layers, sorted_output", [(1, False), (1, True), (3, False)])
def test_lower_thresholds_with_few_rows(layers, sorted_output):
    """Thresholds below the largest table's capacity, as the autotuner sets
    them, and columns above them of matrices with no more rows than that table
    takes: the thresholds change speed, never results."""
    import paper_2010_08526_amd.batched as Bt
    print(f"case: lower thresholds {layers} {sorted_output}", flush=True)
    rng = np.random.default_rng(layers)
    m = 5000
    A = _csc(m, [rng.choice(m, 60, replace=False) for _ in range(300)], rng, torch.float64)
    B = _csc(300, [rng.choice(300, n, replace=False) for n in (1, 30, 70, 150, 290) * 3], rng, torch.float64)
    Ad, Bd = A.to("cuda"), B.to("cuda")
    P = oracle.spgemm(A, B)
    Bt.set_bin_caps(1, (24, 96, 384, 1536, 3840))
    try:
        C = S.spgemm(Ad, Bd, layers=layers, sorted_output=sorted_output)
        order = np.lexsort((C.rowidx.cpu().numpy(), np.repeat(np.arange(C.ncols), np.diff(P.colptr))))
        assert np.diff(P.colptr).max() > 3840
        assert np.array_equal(C.rowidx.cpu().numpy()[order], P.rowidx)
        assert np.array_equal(C.values.cpu().numpy()[order], P.values)
        got = S.masked_xty(Ad, C, Bd)
        D = oracle.Mat(m, C.ncols, P.colptr, C.rowidx.cpu().numpy(), C.values.cpu().numpy())
        assert np.array_equal(got.cpu().numpy(), oracle.masked_xty(A, D, B))
        eng = Bt.BatchedEngine(Ad, Bd)
        eng.forward()
        eng.check()
        assert np.array_equal(eng.values.sort()[0].cpu().numpy(), np.sort(P.values))
    finally:
        Bt.set_bin_caps(1, None)
