"""GPU parity of the pruning that reads each column once: limits of k and of
the list, ties by the thousand (left to the digit kernels), special values,
and columns shorter than k among longer ones.  Bit-exact against the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import host_sorted

pytestmark = pytest.mark.gpu

S = None


def setup_module(module):
    global S
    import paper_2010_08526_amd as lib
    S = lib
    assert torch.cuda.is_available()


def _values(kind, n, rng):
    if kind == "normal":
        return rng.standard_normal(n)
    if kind == "rising":  # every step raises the bound
        return np.arange(n) / 7.0 - 5.0
    if kind == "falling":
        return 5.0 - np.arange(n) / 7.0
    if kind == "levels":
        return rng.integers(-3, 4, n) / 4.0
    if kind == "few_large":
        v = rng.random(n)
        v[-max(1, n // 50):] += 2.0
        return v
    if kind == "equal":
        return np.full(n, 0.5)
    v = rng.standard_normal(n)  # special
    s = rng.random(n)
    v[s < 0.1] = np.nan
    v[(s >= 0.1) & (s < 0.15)] = np.inf
    v[(s >= 0.15) & (s < 0.2)] = -np.inf
    v[(s >= 0.2) & (s < 0.3)] = -0.0
    v[(s >= 0.3) & (s < 0.4)] = 0.0
    return v


@pytest.mark.parametrize("kind", ["normal", "rising", "falling", "levels", "few_large", "equal", "special"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_prune_once(kind, dtype):
    print(f"case: prune once {kind} {dtype}", flush=True)
    rng = np.random.default_rng(len(kind))
    lens = [0, 1, 2, 255, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 2560, 2561, 4097, 9000, 30011]
    m = 40000
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ri = np.concatenate([rng.choice(m, n, replace=False) for n in lens]).astype(np.int32)
    v = torch.from_numpy(np.concatenate([_values(kind, n, rng) for n in lens])).to(dtype)
    M = synth.CSC(m, len(lens), torch.from_numpy(cp), torch.from_numpy(ri), v)
    D = M.to("cuda")
    assert 1025 <= M.nnz // len(lens)  # (so every k below takes the kernel, up to its limit)
    for k in (1, 2, 100, 512, 513, 1024, 1025):
        for thr in (-np.inf, 0.0, 0.1, 1e300, np.nan):
            G = S.prune_topk(D, thr, k)
            P = oracle.prune_topk(M, thr, k)
            cp_, ri_, v_ = host_sorted(G)
            what = f"{kind} k={k} thr={thr}"
            assert np.array_equal(G.colptr.cpu().numpy(), P.colptr), what
            assert np.array_equal(G.rowidx.cpu().numpy(), P.rowidx), what  # input order
            assert np.array_equal(G.values.double().cpu().numpy(), P.values.astype(np.float64)), what


@pytest.mark.parametrize("kind", ["normal", "rising", "falling", "levels", "few_large", "equal", "special"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_prune_once_among_long_columns(kind, dtype):
    """Columns long enough on average for the one reading up to its largest k,
    lists of both sizes; short columns, and ones shorter than k, among them."""
    print(f"case: prune once long {kind} {dtype}", flush=True)
    rng = np.random.default_rng(len(kind) + 7)
    lens = [0, 1, 300, 339, 341, 343, 511, 513, 959, 961, 1023, 1025, 2047, 2048, 2049, 3000, 9000, 60011, 300007]
    m = 400000
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ri = np.concatenate([rng.choice(m, n, replace=False) for n in lens]).astype(np.int32)
    v = torch.from_numpy(np.concatenate([_values(kind, n, rng) for n in lens])).to(dtype)
    M = synth.CSC(m, len(lens), torch.from_numpy(cp), torch.from_numpy(ri), v)
    D = M.to("cuda")
    assert 16 * 960 <= M.nnz // len(lens)
    for k, thr in ((1, -np.inf), (340, 0.0), (341, -np.inf), (342, 0.1), (600, -np.inf), (960, 0.0), (961, 0.0)):
        G = S.prune_topk(D, thr, k)
        P = oracle.prune_topk(M, thr, k)
        what = f"{kind} k={k} thr={thr}"
        assert np.array_equal(G.colptr.cpu().numpy(), P.colptr), what
        assert np.array_equal(G.rowidx.cpu().numpy(), P.rowidx), what  # input order
        assert np.array_equal(G.values.double().cpu().numpy(), P.values.astype(np.float64)), what


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("lens, k", [(100, 100), (100, 10), (5, 5), (5, 1)])
def test_prune_once_of_many_short_columns(dtype, lens, k):
    """Enough short columns for the one reading; ties by the dozen."""
    print(f"case: prune once short {lens} {k} {dtype}", flush=True)
    rng = np.random.default_rng(lens + k)
    n, m = 9000, 70001
    ln = np.maximum(rng.integers(lens - 2, lens + 6, n), 0)
    cp = np.concatenate([[0], np.cumsum(ln)]).astype(np.int64)
    ri = np.concatenate([rng.choice(m, c, replace=False) for c in ln]).astype(np.int32)
    v = torch.from_numpy(rng.integers(0, 6, ri.size) / 4.0).to(dtype)
    M = synth.CSC(m, n, torch.from_numpy(cp), torch.from_numpy(ri), v)
    assert k <= M.nnz // n
    G, P = S.prune_topk(M.to("cuda"), 0.25, k), oracle.prune_topk(M, 0.25, k)
    assert np.array_equal(G.colptr.cpu().numpy(), P.colptr)
    assert np.array_equal(G.rowidx.cpu().numpy(), P.rowidx)
    assert np.array_equal(G.values.double().cpu().numpy(), P.values.astype(np.float64))


def test_prune_once_reports_a_repeated_row():
    """Two equal entries of one row at the cut."""
    print("case: prune once repeated row", flush=True)
    n = 3000
    r = torch.randperm(5000)[:n].to(torch.int32)
    v = torch.rand(n)
    order = torch.argsort(v, descending=True)
    v[order[9]] = v[order[10]]
    r[order[9]] = r[order[10]]
    C = S.CSC(5000, 1, torch.tensor([0, n], device="cuda"), r.cuda(), v.cuda())
    with pytest.raises(S.SpgemmError):
        S.prune_topk(C, 0.0, 10)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_prune_once_keeps_the_first_of_repeated_rows(dtype):
    """Columns with one row 384 times at the cut and 64 larger entries after
    them, in slots of another wave that has nothing before: reported, and of the
    entries at or above the cut the first k are kept, in input order."""
    import ctypes
    print(f"case: prune once first k {dtype}", flush=True)
    n, k, cols = 2048, 200, 50
    slot, thread = torch.arange(n) // 256, torch.arange(n) % 256
    again = (thread < 64) & (slot < 6)
    larger = (thread >= 192) & (slot == 7)
    r = torch.where(again, 0, 1 + torch.arange(n)).to(torch.int32).repeat(cols).cuda()
    v = torch.where(again, 1.0, torch.where(larger, 2.0, -1.0)).to(dtype).repeat(cols).cuda()
    # (and one long column, by which the columns are long enough on average)
    long = 400000
    r = torch.cat([r, torch.arange(long, dtype=torch.int32, device="cuda")])
    v = torch.cat([v, torch.arange(long, device="cuda").to(dtype)])
    cp = torch.cat([torch.arange(0, n * cols + 1, n), torch.tensor([n * cols + long])])
    cols += 1
    C = S.CSC(long, cols, cp.cuda(), r, v)
    out = (torch.empty(cols + 1, dtype=torch.int64, device="cuda"),
           torch.empty(k * cols, dtype=torch.int32, device="cuda"), torch.empty(k * cols, dtype=dtype, device="cuda"))
    ws = S.alloc_workspace(S.workspace_size(S.OP_PRUNE, C))
    S._check(S._lib.spgemm_prune_topk(ctypes.byref(S.desc(C)), 0.0, k, *[S._ptr(x) for x in out], k * cols, S._ptr(ws),
                                      ws.numel(), S._stream(None)), "prune")
    assert S.ws_status_code(ws) == (S.E_DEVICE, 10)
    assert torch.equal(out[0].cpu(), torch.arange(0, k * cols + 1, k))
    assert torch.all(out[1][:-k] == 0) and torch.all(out[2][:-k] == 1.0)
    assert torch.equal(out[1][-k:].cpu(), torch.arange(long - k, long, dtype=torch.int32))


def test_prune_once_in_a_graph():
    print("case: prune once graph", flush=True)
    rng = np.random.default_rng(3)
    lens = rng.integers(0, 6000, 300)
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ri = np.concatenate([rng.choice(7000, n, replace=False) for n in lens]).astype(np.int32)
    M = synth.CSC(7000, 300, torch.from_numpy(cp), torch.from_numpy(ri), torch.from_numpy(rng.random(ri.size)).float())
    D = M.to("cuda")
    k, cap = 50, 50 * 300
    out = (torch.empty(301, dtype=torch.int64, device="cuda"), torch.empty(cap, dtype=torch.int32, device="cuda"),
           torch.empty(cap, device="cuda"))
    ws = S.alloc_workspace(S.workspace_size(S.OP_PRUNE, D))
    import ctypes

    def call():
        S._check(S._lib.spgemm_prune_topk(ctypes.byref(S.desc(D)), 0.2, k, *[S._ptr(x) for x in out], cap, S._ptr(ws),
                                          ws.numel(), S._stream(None)), "prune")

    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        call()
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for _ in range(4):
        D.values.copy_(torch.rand_like(D.values))  # eager work between replays
        for x in out:
            x.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        S.check_ws(ws)
        P = oracle.prune_topk(synth.CSC(7000, 300, M.colptr, M.rowidx, D.values.cpu()), 0.2, k)
        n = int(out[0][-1])
        assert np.array_equal(out[0].cpu().numpy(), P.colptr)
        assert np.array_equal(out[1][:n].cpu().numpy(), P.rowidx)
        assert np.array_equal(out[2][:n].double().cpu().numpy(), P.values.astype(np.float64))


def test_many_short_columns_in_a_graph():
    """The one reading over many short columns, and a sort of few columns, both
    captured and replayed over new values and rows."""
    import ctypes
    print("case: prune short and sort few in a graph", flush=True)
    rng = np.random.default_rng(9)
    n, m, k = 9000, 5000, 5
    lens = rng.integers(10, 40, n)
    cp = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ri = np.concatenate([rng.choice(m, c, replace=False) for c in lens]).astype(np.int32)
    M = synth.CSC(m, n, torch.from_numpy(cp), torch.from_numpy(ri), torch.from_numpy(rng.random(ri.size)).float())
    D = M.to("cuda")
    few = S.CSC(m, 300, D.colptr[:301], D.rowidx[:int(cp[300])], D.values[:int(cp[300])])
    out = (torch.empty(n + 1, dtype=torch.int64, device="cuda"),
           torch.empty(k * n, dtype=torch.int32, device="cuda"), torch.empty(k * n, device="cuda"))
    srt = (torch.empty_like(few.rowidx), torch.empty_like(few.values))
    ws = S.alloc_workspace(S.workspace_size(S.OP_PRUNE, D))
    ws2 = S.alloc_workspace(S.workspace_size(S.OP_SORT, few))

    def call():
        S._check(S._lib.spgemm_prune_topk(ctypes.byref(S.desc(D)), 0.2, k, *[S._ptr(x) for x in out], k * n,
                                          S._ptr(ws), ws.numel(), S._stream(None)), "prune")
        S.sort_columns(few, *srt, ws=ws2)

    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        call()
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    col = np.repeat(np.arange(300), lens[:300])
    for i in range(4):
        D.values.copy_(torch.rand_like(D.values))  # eager work between replays
        D.rowidx.copy_(torch.remainder(D.rowidx + 1 + i, m))
        for x in out + srt:
            x.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        S.check_many([ws, ws2])
        H = synth.CSC(m, n, M.colptr, D.rowidx.cpu(), D.values.cpu())
        P = oracle.prune_topk(H, 0.2, k)
        assert np.array_equal(out[0].cpu().numpy(), P.colptr)
        kept = int(out[0][-1])
        assert np.array_equal(out[1][:kept].cpu().numpy(), P.rowidx)
        assert np.array_equal(out[2][:kept].double().cpu().numpy(), P.values.astype(np.float64))
        r, v = H.rowidx.numpy()[:col.size], H.values.numpy()[:col.size]
        order = np.lexsort((r, col))
        assert np.array_equal(srt[0].cpu().numpy(), r[order]) and np.array_equal(srt[1].cpu().numpy(), v[order])
