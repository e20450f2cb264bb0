"""Products and gradients on streams given as torch streams or as handles:
what is read back or refreshed belongs to the call that it was asked of."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import synth
from tests.gpu_util import assert_matches

pytestmark = pytest.mark.gpu

S = None


def setup_module(module):
    global S
    import paper_2010_08526_amd as lib
    S = lib
    assert torch.cuda.is_available()


def test_context_is_the_stream():
    print("case: stream contexts", flush=True)
    side = torch.cuda.Stream()
    for h in (0, int(side.cuda_stream), side):
        with S._on_stream(h):
            assert int(torch.cuda.current_stream().cuda_stream) == S._stream(h)
        with torch.cuda.stream(side), S._on_stream(h):
            assert int(torch.cuda.current_stream().cuda_stream) == S._stream(h)


def test_counts_of_each_run():
    """The counts of a run on the default stream are that run's, also when
    they are read after the engine's next run."""
    print("case: counts of each run", flush=True)
    A = synth.erdos_renyi(40000, 40000, 3, 5, torch.float32)
    B = synth.erdos_renyi(40000, 40000, 5, 6, torch.float32)
    B2 = synth.erdos_renyi(40000, 40000, 5, 7, torch.float32)
    eng = S.Engine(A.to("cuda"), B.to("cuda"))
    _, plan = eng.run()
    eng.B.rowidx.copy_(B2.rowidx)
    _, plan2 = eng.run()
    assert np.array_equal(plan.nnz_host[0], oracle.count(A, B))
    assert np.array_equal(plan2.nnz_host[0], oracle.count(A, synth.CSC(B.nrows, B.ncols, B.colptr, B2.rowidx,
                                                                       B.values)))


def test_refresh_on_the_default_stream_by_handle():
    print("case: refresh by handle 0", flush=True)
    A = synth.erdos_renyi(500, 500, 6, 5, torch.float64).to("cuda")
    B = synth.erdos_renyi(500, 500, 5, 6, torch.float64).to("cuda")
    C = S.spgemm(A, B)
    dC = torch.ones_like(C.values)
    bw = S.Backward(A, B, C, stream=0)
    dA, _ = bw(dC)
    B2 = S.CSC(B.nrows, B.ncols, B.colptr, B.rowidx, B.values * 2)
    bw.refresh_values(B2, stream=0)
    dA2, _ = bw(dC)
    bw.check()
    assert torch.allclose(dA2, 2 * dA, rtol=1e-12)


@pytest.mark.parametrize("n", [8000, 40000])
def test_counts_read_on_another_stream(n):
    """A plan made on a busy side stream, its counts read on the default one
    at once."""
    print(f"case: counts on another stream {n}", flush=True)
    A = synth.erdos_renyi(n, n, 3, 5, torch.float32)
    B = synth.erdos_renyi(n, n, 5, 6, torch.float32)
    eng = S.Engine(A.to("cuda"), B.to("cuda"))
    side = torch.cuda.Stream()
    want = oracle.count(A, B)
    torch.cuda.synchronize()
    for stream in (side, int(side.cuda_stream)):
        eng.nnz.zero_()
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            torch.cuda._sleep(10_000_000)
        plan = eng.plan(stream)
        assert np.array_equal(plan.nnz_host[0], want) and plan.total_flops == 15 * n


def test_output_memory_in_use_on_another_stream():
    """A product on a side stream whose output takes memory that the default
    stream, behind a long kernel, has yet to write to."""
    print("case: output memory in use", flush=True)
    A = synth.erdos_renyi(20000, 20000, 6, 5, torch.float64)
    eng = S.Engine(A.to("cuda"), A.to("cuda"))
    side = torch.cuda.Stream()
    want, _ = eng.run(stream=side)
    torch.cuda.synchronize()
    n = want.nnz
    x = [torch.empty(n, dtype=torch.float64, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")]
    torch.cuda._sleep(10_000_000)
    for t in x:
        t.fill_(7)
    del x, t
    C, _ = eng.run(stream=side)
    torch.cuda.synchronize()
    assert torch.equal(C.colptr, want.colptr)
    assert_matches(C, oracle.spgemm(A, A), torch.float64, "side stream")
