"""Streams that the binding gives to torch's own work, checked without a GPU:
torch's stream calls are replaced by stand-ins that record what is asked for."""
from __future__ import annotations

import contextlib
import types

import numpy as np
import pytest
import torch

import paper_2010_08526_amd as S


class FakeCuda:
    """Stand-ins for torch.cuda's streams; `entered` lists the handles whose
    context was entered (an external stream of handle 0 is another stream)."""

    def __init__(self, monkeypatch, current):
        self.entered = []
        self.current = current
        self.waits = []  # (stream, the stream it waits for)
        stream = lambda h: types.SimpleNamespace(  # noqa: E731
            cuda_stream=h, wait_stream=lambda o: self.waits.append((h, o.cuda_stream)))
        monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: stream(self.current))
        monkeypatch.setattr(torch.cuda, "default_stream", lambda *a: stream(0))
        monkeypatch.setattr(torch.cuda, "ExternalStream", lambda h: stream(h if h else "another stream"))
        monkeypatch.setattr(torch.cuda, "stream", self.enter)

    @contextlib.contextmanager
    def context(self, s):
        before, self.current = self.current, s.cuda_stream
        yield s
        self.current = before

    def enter(self, s):
        self.entered.append(s.cuda_stream)
        return self.context(s)


@pytest.mark.parametrize("current", [0, 4096])
@pytest.mark.parametrize("handle", [None, 0, 4096, 8192])
def test_context_of_a_handle(monkeypatch, current, handle):
    """The context of a handle is that stream, for handle 0 the default one."""
    fake = FakeCuda(monkeypatch, current)
    S._on_stream(handle)
    used = fake.entered[0] if fake.entered else current
    assert used == (current if handle is None else handle)


class Counts:
    """Stand-in for the counts on the device: notes what is done on which stream."""

    def __init__(self, fake, rows, n):
        self.fake, self.rows, self.n, self.log = fake, rows, n, []

    def data_ptr(self):
        return 0

    def clone(self):
        self.log.append(("clone", self.fake.current))
        return self

    def cpu(self):
        self.log.append(("read", self.fake.current))
        return torch.ones((self.rows, self.n), dtype=torch.int64)


@pytest.mark.parametrize("n", [100, 40000])
@pytest.mark.parametrize("handle", [None, 0, 4096])
def test_counts_are_read_after_the_symbolic_pass(monkeypatch, n, handle):
    """The counts of a plan made on one stream and read on another: read (or
    copied, and read once that is done) where the symbolic pass ran."""
    fake = FakeCuda(monkeypatch, 0)
    counts = Counts(fake, 1, n)

    class Event:
        def record(self, stream=None):
            counts.log.append(("record", fake.current))

        def synchronize(self):
            counts.log.append(("wait", None))

    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(S, "symbolic", lambda *a, **k: None)
    monkeypatch.setattr(S._lib, "spgemm_count_sums_rows", lambda *a: 0)
    eng = object.__new__(S.Engine)
    eng.A = eng.B = S.CSC(100, n, None, torch.zeros(0), None)
    eng.L, eng.vbytes, eng.max_batches, eng.sorted_output = 1, 4, 1 << 16, False
    eng.input_bytes, eng.reserve_bytes, eng.budget_bytes = 0, 0, 1 << 30
    eng.flops = eng.ws_sym = None
    eng.ws_scan = torch.zeros(16)
    eng.nnz = counts
    plan = eng.plan(handle)
    assert np.array_equal(plan.nnz_host, np.ones((1, n)))
    s = handle or 0
    if n < 32768:
        assert counts.log == [("read", s)]
    else:
        assert counts.log == [("clone", s), ("record", s), ("wait", None), ("read", 0)]
    assert plan.nnz_host is plan.nnz_host


@pytest.mark.parametrize("handle", [None, 0, 4096])
@pytest.mark.parametrize("layers", [1, 2])
def test_new_output_waits_for_the_memory(monkeypatch, handle, layers):
    """The first kernel that writes a whole product's output, whose memory is
    the current stream's, comes after that stream's work."""
    fake = FakeCuda(monkeypatch, 0)
    order = []
    monkeypatch.setattr(S, "colptr", lambda *a: order.append(len(fake.waits)))
    monkeypatch.setattr(S, "numeric", lambda *a: order.append(len(fake.waits)))
    monkeypatch.setattr(S, "merge", lambda *a: order.append(len(fake.waits)))
    monkeypatch.setattr(S, "alloc_workspace", lambda *a: torch.zeros(256, dtype=torch.uint8))
    eng = object.__new__(S.Engine)
    eng.A = eng.B = S.CSC(4, 4, None, torch.zeros(0), None)
    eng.L, eng.vbytes, eng.vdtype, eng.sorted_output, eng.semiring = layers, 4, torch.float32, False, 0
    eng.device, eng._bufs = "cpu", {}
    eng.ws_scan = eng.ws_num = eng.ws_mrg = eng.flops = torch.zeros(16)
    rows = layers + 1 if layers > 1 else 1
    eng.nnz = torch.ones((rows, 4), dtype=torch.int64)
    plan = types.SimpleNamespace(batch_nnz=np.full((1, rows), 4), nbatches=1, bounds=[0, 4], longest=1, row_longest=None)
    eng._whole(plan, handle)
    assert fake.waits == ([(4096, 0)] if handle == 4096 else [])
    assert order and set(order) == {len(fake.waits)}


@pytest.mark.parametrize("handle", [None, 0, 4096])
def test_gradient_memory_is_the_current_streams(monkeypatch, handle):
    """What a Backward keeps is used, and given back, on any stream: it is not
    taken from the pool of the stream that fills it; the fill waits for it."""
    fake = FakeCuda(monkeypatch, 0)
    pools, fills = [], []

    class Values(torch.Tensor):
        @classmethod
        def __torch_function__(cls, func, types, args=(), kwargs=None):
            name = func.__name__
            if name in ("clone", "empty_like"):
                pools.append(fake.current)
            if name in ("clone", "copy_"):
                fills.append((fake.current, len(fake.waits)))
            return super().__torch_function__(func, types, args, kwargs or {})

    def workspace(nbytes, device=None):
        pools.append(fake.current)
        return torch.zeros(256, dtype=torch.uint8)

    monkeypatch.setattr(S, "alloc_workspace", workspace)
    cp, ri = torch.arange(5), torch.arange(4, dtype=torch.int32)
    M = S.CSC(4, 4, cp, ri, torch.ones(4).as_subclass(Values))
    bw = S.Backward(M, M, M, stream=handle)
    assert bw.ws_f is not None and torch.equal(torch.Tensor(bw._b), torch.ones(4))
    assert pools == [0, 0]
    assert fills == [(handle or 0, 1 if handle else 0)]


@pytest.mark.parametrize("handle", [None, 0, 4096])
def test_longest_row_waits_for_its_workspace(monkeypatch, handle):
    fake = FakeCuda(monkeypatch, 0)
    waited = []
    monkeypatch.setattr(S, "alloc_workspace", lambda *a: torch.zeros(256, dtype=torch.uint8))
    monkeypatch.setattr(S._lib, "spgemm_longest_row", lambda *a: waited.append(len(fake.waits)) or 0)
    S._longest_row(S.CSC(4, 4, torch.arange(5), torch.arange(4, dtype=torch.int32), None), handle)
    assert waited == [1 if handle else 0]
