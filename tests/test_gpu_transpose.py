"""GPU parity of the transpose: columns against the tiles of 4096 entries it
works on (empty runs longer than a tile's threads, columns longer than a tile,
starts at tile edges), every output it can be asked for."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

S = None


def setup_module(module):
    global S
    import paper_2010_08526_amd as lib
    S = lib
    assert torch.cuda.is_available()


LENS = {
    "one": [1], "empty": [0, 0, 0], "pairs": [2] * 9001, "edge": [4096, 4096, 1], "edge1": [4095, 2, 4095],
    "long": [3, 20000, 0, 1], "gaps": [1] + [0] * 70000 + [5] + [0] * 300 + [4090] + [0] * 9000 + [7],
    "ragged": None,
}


@pytest.mark.parametrize("case", sorted(LENS))
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_transpose_tiles(case, dtype):
    print(f"case: transpose {case} {dtype}", flush=True)
    rng = np.random.default_rng(len(case))
    m = 30000
    lens = np.array(LENS[case] if LENS[case] is not None else rng.integers(0, 300, 2000))
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ri = np.concatenate([rng.choice(m, n, replace=False) for n in lens]).astype(np.int32)
    v = torch.from_numpy(rng.standard_normal(ri.size)).to(dtype)
    X = S.CSC(m, lens.size, torch.from_numpy(cp).cuda(), torch.from_numpy(ri).cuda(), v.cuda())
    col = np.repeat(np.arange(lens.size), lens)
    want = np.lexsort((col, ri))  # by row, then column
    for values, perm in ((True, True), (True, False), (False, True), (False, False)):
        ws = S.alloc_workspace(S.workspace_size(S.OP_TRANSPOSE, X))
        T, pm = S.transpose(X, ws, values=values, perm=perm)
        S.check_ws(ws)
        tcp = T.colptr.cpu().numpy()
        assert np.array_equal(tcp, np.concatenate([[0], np.cumsum(np.bincount(ri, minlength=m))]))
        tri = T.rowidx.cpu().numpy()
        order = np.lexsort((tri, np.repeat(np.arange(m), np.diff(tcp))))
        assert np.array_equal(tri[order], col[want])
        if values:
            assert np.array_equal(T.values.cpu().numpy()[order], v.numpy()[want])
        if perm:
            assert np.array_equal(pm.cpu().numpy()[order], want)


@pytest.mark.parametrize("span", [8191, 8192, 8193, 8194, 16385, 300000])
@pytest.mark.parametrize("nnz", [2, 5, 4096, 4097, 9000])
def test_transpose_of_mostly_empty_columns(span, nnz):
    """Entries spread over `span` columns between empty ones, the first and the
    last of them not empty, some of several entries: tiles on both sides of the
    span from which entries look their columns up."""
    print(f"case: transpose span {span} nnz {nnz}", flush=True)
    rng = np.random.default_rng(span + nnz)
    m, before, after = 20000, 700, 9001
    n = before + span + after
    at = np.concatenate([[0, span - 1], rng.integers(0, span, nnz - 2)])
    lens = np.bincount(before + at, minlength=n)
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ri = np.concatenate([rng.choice(m, c, replace=False) for c in lens[lens > 0]]).astype(np.int32)
    v = rng.standard_normal(nnz)
    X = S.CSC(m, n, torch.from_numpy(cp).cuda(), torch.from_numpy(ri).cuda(), torch.from_numpy(v).cuda())
    ws = S.alloc_workspace(S.workspace_size(S.OP_TRANSPOSE, X))
    T, pm = S.transpose(X, ws)
    S.check_ws(ws)
    col = np.repeat(np.arange(n), lens)
    want = np.lexsort((col, ri))
    tcp, tri = T.colptr.cpu().numpy(), T.rowidx.cpu().numpy()
    assert np.array_equal(tcp, np.concatenate([[0], np.cumsum(np.bincount(ri, minlength=m))]))
    order = np.lexsort((tri, np.repeat(np.arange(m), np.diff(tcp))))
    assert np.array_equal(tri[order], col[want])
    assert np.array_equal(T.values.cpu().numpy()[order], v[want])
    assert np.array_equal(pm.cpu().numpy()[order], want)


def test_transpose_reports_a_bad_row():
    print("case: transpose bad row", flush=True)
    X = S.CSC(5, 2, torch.tensor([0, 2, 3], device="cuda"), torch.tensor([1, 7, 2], dtype=torch.int32, device="cuda"),
              torch.ones(3, device="cuda"))
    ws = S.alloc_workspace(S.workspace_size(S.OP_TRANSPOSE, X))
    S.transpose(X, ws)
    with pytest.raises(S.SpgemmError):
        S.check_ws(ws)


@pytest.mark.parametrize("m, n, nnz", [(1, 1, 1), (5, 0, 0), (0, 3, 0), (7, 4000, 9000), (100000, 300, 20000)])
def test_longest_row(m, n, nnz):
    print(f"case: longest row {m} {n} {nnz}", flush=True)
    rng = np.random.default_rng(nnz)
    at = rng.choice(m * n, nnz, replace=False) if nnz else np.zeros(0, int)
    at.sort()
    lens = np.bincount(at // max(m, 1), minlength=n)
    X = S.CSC(m, n, torch.from_numpy(np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)).cuda(),
              torch.from_numpy((at % max(m, 1)).astype(np.int32)).cuda(), None)
    assert S._longest_row(X) == np.bincount(at % max(m, 1), minlength=1).max()
