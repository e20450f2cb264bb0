"""Python binding of libspgemm (the C ABI in include/spgemm.h).

Argument marshalling only: every step of the product runs in the library's
HIP kernels or its host-side planner.  torch supplies device memory and
streams.  torch is imported before the library is loaded so that both use
one HIP runtime.  There is no fallback: if the library is missing the
import fails.
"""
from __future__ import annotations

import contextlib
import ctypes
import os
from dataclasses import dataclass

import numpy as np
import torch

_PKG = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_PKG, "_lib", "libspgemm.so")

if not os.path.exists(LIB_PATH):
    raise ImportError(f"{LIB_PATH} is missing; build it with `python paper_2010_08526_amd/build.py`")
_lib = ctypes.CDLL(LIB_PATH)

# ---------------------------------------------------------------- constants
OK, E_INVAL, E_SHAPE, E_DTYPE, E_BUDGET, E_WORKSPACE, E_HIP, E_OVERFLOW, E_DEVICE = 0, -1, -2, -3, -4, -5, -6, -7, -8
F32, F64 = 0, 1
# semirings of the numeric pass and the merge (spgemm_semiring)
PLUS_TIMES, MIN_PLUS, OR_AND = 0, 1, 2
SEMIRINGS = {"plus_times": PLUS_TIMES, "min_plus": MIN_PLUS, "or_and": OR_AND}
(OP_SYMBOLIC, OP_NUMERIC, OP_MERGE, OP_COLPTR, OP_MASKED_XTY, OP_TRANSPOSE, OP_BATCHED_FORWARD, OP_BATCHED_BACKWARD,
 OP_PRUNE, OP_SORT) = range(10)
MAX_PARTS = 4096

_DTYPE = {torch.float32: F32, torch.float64: F64}


class spgemm_csc(ctypes.Structure):
    _fields_ = [("nrows", ctypes.c_int64), ("ncols", ctypes.c_int64), ("nnz", ctypes.c_int64),
                ("colptr", ctypes.c_void_p), ("rowidx", ctypes.c_void_p), ("values", ctypes.c_void_p),
                ("dtype", ctypes.c_int32)]


_P = ctypes.POINTER(spgemm_csc)
_vp, _i64, _i32, _sz = ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_size_t

_lib.spgemm_workspace_size.argtypes = [ctypes.c_int, _P, _P, _i64, _i64, _i32, ctypes.POINTER(_sz)]
_lib.spgemm_symbolic.argtypes = [_P, _P, _i64, _i64, _i32, _vp, _vp, _vp, _sz, _vp]
_lib.spgemm_plan_batches.argtypes = [_vp, _i64, _i32, _i32, ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint64, _i32,
                                     _vp, ctypes.POINTER(_i32), _vp]
_lib.spgemm_colptr.argtypes = [_vp, _i64, _vp, _vp, _sz, _vp]
_lib.spgemm_numeric.argtypes = [_P, _P, _i64, _i64, _i32, _i32, _vp, _vp, _vp, _vp, _i32, _vp, _sz, _vp]
_lib.spgemm_merge.argtypes = [_P, _i32, _vp, _vp, _vp, _i32, _vp, _sz, _vp]
_lib.spgemm_ws_status.argtypes = [_vp, _vp]
_lib.spgemm_ws_status_code.argtypes = [_vp, _vp, _vp]
_lib.spgemm_ws_invalidate.argtypes = [_vp, _vp]
_lib.spgemm_batched_forward.argtypes = [_P, _P, _i64, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]
_lib.spgemm_batched_masked_xty.argtypes = [_P, _P, _P, _vp, _vp, _sz, _vp]
_lib.spgemm_batched_backward.argtypes = [_P, _P, _P, _vp, _vp, _vp, _vp, _sz, _vp]
_lib.spgemm_set_bin_caps.argtypes = [_i32, _vp]
_lib.spgemm_batch_pack.argtypes = [_P, _i32, _vp, _vp, _vp, _vp, _vp, _sz, _vp]
_lib.spgemm_debug_min_bin.argtypes = [_i32]
_lib.spgemm_profile_enable.argtypes = [_i32]
_lib.spgemm_profile_report.argtypes = [ctypes.c_char_p, _sz]


def profile_enable(on: bool = True):
    """Start (or stop) per-kernel HIP-event timing inside the library."""
    _check(_lib.spgemm_profile_enable(int(on)), "spgemm_profile_enable")


def profile_report() -> dict:
    """{kernel name: (total ms, launches)} since profile_enable(True)."""
    buf = ctypes.create_string_buffer(1 << 16)
    _check(_lib.spgemm_profile_report(buf, len(buf)), "spgemm_profile_report")
    out = {}
    for line in buf.value.decode().splitlines():
        name, ms, cnt = line.split()
        out[name] = (float(ms), int(cnt))
    return out
_lib.spgemm_status_string.restype = ctypes.c_char_p
_lib.spgemm_status_string.argtypes = [ctypes.c_int]
_lib.spgemm_last_hip_error.restype = ctypes.c_int


class SpgemmError(RuntimeError):
    def __init__(self, status: int, where: str = ""):
        self.status = status
        msg = status_string(status)
        if status == E_HIP:
            msg += f" (hipError {int(_lib.spgemm_last_hip_error())})"
        super().__init__(f"{where}: {msg}" if where else msg)


def status_string(status: int) -> str:
    return _lib.spgemm_status_string(int(status)).decode()


def _check(rc: int, where: str):
    if rc != OK:
        raise SpgemmError(rc, where)


def _ptr(t) -> int | None:
    """Address of a tensor (or an address as it is)."""
    return t if t is None or isinstance(t, int) else t.data_ptr()


def _stream(stream) -> int | None:
    if stream is None:
        return int(torch.cuda.current_stream().cuda_stream) if torch.cuda.is_available() else None
    return int(getattr(stream, "cuda_stream", stream))


@dataclass
class CSC:
    """A CSC matrix in torch tensors: colptr int64[ncols+1], rowidx int32[nnz],
    values float32/float64[nnz] (or None)."""

    nrows: int
    ncols: int
    colptr: torch.Tensor
    rowidx: torch.Tensor
    values: torch.Tensor | None

    @property
    def nnz(self) -> int:
        return int(self.rowidx.numel())


def desc(M, dtype: int | None = None) -> spgemm_csc:
    """C descriptor of any object with nrows/ncols/colptr/rowidx/values."""
    if isinstance(M, spgemm_csc):
        return M
    v = M.values
    if dtype is None:
        dtype = _DTYPE.get(v.dtype, -1) if v is not None else F32
    return spgemm_csc(int(M.nrows), int(M.ncols), int(M.rowidx.numel()), _ptr(M.colptr), _ptr(M.rowidx), _ptr(v),
                      int(dtype))


# ------------------------------------------------------------ thin wrappers
def workspace_size(op: int, A=None, B=None, c0: int = 0, c1: int = 0, n_layers: int = 1) -> int:
    out = _sz(0)
    a = ctypes.byref(desc(A)) if A is not None else None
    b = ctypes.byref(desc(B)) if B is not None else None
    _check(_lib.spgemm_workspace_size(op, a, b, c0, c1, n_layers, ctypes.byref(out)), "spgemm_workspace_size")
    return int(out.value)


def alloc_workspace(nbytes: int, device=None) -> torch.Tensor:
    """A 256-byte aligned device buffer (torch's allocator aligns to 512)."""
    t = torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=device or "cuda")
    assert t.data_ptr() % 256 == 0
    t[:4096].zero_()  # header: no status recorded before the first call
    return t


def symbolic(A, B, c0: int, c1: int, n_layers: int, flops_out, nnz_out, ws: torch.Tensor, stream=None):
    _check(_lib.spgemm_symbolic(ctypes.byref(desc(A)), ctypes.byref(desc(B)), c0, c1, n_layers, _ptr(flops_out),
                                _ptr(nnz_out), _ptr(ws), ws.numel(), _stream(stream)), "spgemm_symbolic")


def plan_batches(nnz_host, ncols: int, n_layers: int, value_bytes: int, input_bytes: int, budget_bytes: int,
                 reserve_bytes: int = 0, max_batches: int = 1 << 16):
    """Returns (bounds: list[int], batch_nnz: np.ndarray[b, rows])."""
    nnz_host = np.ascontiguousarray(np.asarray(nnz_host, dtype=np.int64))
    rows = n_layers + 1 if n_layers > 1 else 1
    max_batches = min(max_batches, max(1, ncols))  # a batch holds at least one column
    bounds = np.zeros(max(1, max_batches) + 1, np.int64)
    tot = np.zeros(max(1, max_batches) * rows, np.int64)
    nb = _i32(0)
    _check(_lib.spgemm_plan_batches(nnz_host.ctypes.data, ncols, n_layers, value_bytes, int(input_bytes),
                                    int(budget_bytes), int(reserve_bytes), max_batches, bounds.ctypes.data,
                                    ctypes.byref(nb), tot.ctypes.data), "spgemm_plan_batches")
    b = int(nb.value)
    return bounds[:b + 1].tolist(), tot[:b * rows].reshape(b, rows)


def colptr(counts: torch.Tensor, out: torch.Tensor, ws: torch.Tensor, stream=None):
    n = counts.numel()
    _check(_lib.spgemm_colptr(_ptr(counts), n, _ptr(out), _ptr(ws), ws.numel(), _stream(stream)), "spgemm_colptr")


def semiring_id(semiring) -> int:
    """spgemm_semiring value of a name ('plus_times', 'min_plus', 'or_and') or id."""
    if isinstance(semiring, str):
        if semiring not in SEMIRINGS:
            raise ValueError(f"unknown semiring {semiring!r}")
        return SEMIRINGS[semiring]
    return int(semiring)


NO_BOUND = (1 << 63) - 1  # max_len of a caller that knows no bound on the columns' entries


def numeric(A, B, c0: int, c1: int, layer: int, n_layers: int, flops, c_colptr, c_rowidx, c_values,
            ws: torch.Tensor, stream=None, semiring=PLUS_TIMES, max_len: int = NO_BOUND):
    _check(_lib.spgemm_numeric_upto(ctypes.byref(desc(A)), ctypes.byref(desc(B)), c0, c1, layer, n_layers,
                                    _ptr(flops), _ptr(c_colptr), _ptr(c_rowidx), _ptr(c_values),
                                    semiring_id(semiring), max_len, _ptr(ws), ws.numel(), _stream(stream)),
           "spgemm_numeric")


COUNT_SUMS_MAX_ROWS = 64
SLAB_MIN_ROWS = 5120  # more rows than this: heavy columns are formed from a slabbed copy of A
_lib.spgemm_count_sums_rows.argtypes = [_vp, _i64, _i32, _vp, _vp, _vp, _sz, _vp]
_lib.spgemm_numeric_upto.argtypes = [_P, _P, _i64, _i64, _i32, _i32, _vp, _vp, _vp, _vp, _i32, _i64, _vp, _sz, _vp]
_lib.spgemm_numeric_sorted.argtypes = [_P, _P, _i64, _i64, _vp, _vp, _vp, _vp, _vp, _vp, ctypes.c_double, _i32, _vp,
                                       _sz, _vp]
_lib.spgemm_numeric_sorted_upto.argtypes = [_P, _P, _i64, _i64, _vp, _vp, _vp, _vp, _vp, _vp, ctypes.c_double, _i32,
                                            _i64, _vp, _sz, _vp]

# Compression ratio up to which a column of at most 4096 product terms is
# formed in row order by expand-sort-compress rather than hashed and sorted.
ESC_CF_DEFAULT = 2.0


def numeric_sorted(A, B, c0: int, c1: int, flops, c_colptr, c_rowidx, c_values, tmp_rowidx, tmp_values,
                   ws: torch.Tensor, stream=None, semiring=PLUS_TIMES, esc_cf: float = ESC_CF_DEFAULT,
                   max_len: int = NO_BOUND):
    """Columns [c0, c1) of A*B in row order: low-compression columns by
    expand-sort-compress, the others hashed into tmp_* and sorted."""
    _check(_lib.spgemm_numeric_sorted_upto(ctypes.byref(desc(A)), ctypes.byref(desc(B)), c0, c1, _ptr(flops),
                                           _ptr(c_colptr), _ptr(c_rowidx), _ptr(c_values), _ptr(tmp_rowidx),
                                           _ptr(tmp_values), float(esc_cf), semiring_id(semiring), max_len, _ptr(ws),
                                           ws.numel(), _stream(stream)), "spgemm_numeric_sorted")


def merge(parts, c_colptr, c_rowidx, c_values, ws: torch.Tensor, stream=None, semiring=PLUS_TIMES):
    arr = (spgemm_csc * len(parts))(*[desc(p) for p in parts])
    _check(_lib.spgemm_merge(arr, len(parts), _ptr(c_colptr), _ptr(c_rowidx), _ptr(c_values), semiring_id(semiring),
                             _ptr(ws), ws.numel(), _stream(stream)), "spgemm_merge")


_lib.spgemm_sort_columns.argtypes = [_P, _vp, _vp, _vp, _sz, _vp]


def sort_columns(C, rowidx_out: torch.Tensor | None = None, values_out: torch.Tensor | None = None,
                 ws: torch.Tensor | None = None, stream=None) -> CSC:
    """C with every column's entries in row order (values moved with their
    rows), written to separate arrays; C's column pointers are shared."""
    dev = C.rowidx.device
    n = C.nnz
    if ws is None:
        ws = alloc_workspace(workspace_size(OP_SORT, C), dev)
    if rowidx_out is None:
        rowidx_out = torch.empty(max(1, n), dtype=torch.int32, device=dev)
    if values_out is None:
        values_out = torch.empty(max(1, n), dtype=C.values.dtype, device=dev)
    _check(_lib.spgemm_sort_columns(ctypes.byref(desc(C)), _ptr(rowidx_out), _ptr(values_out), _ptr(ws), ws.numel(),
                                    _stream(stream)), "spgemm_sort_columns")
    return CSC(C.nrows, C.ncols, C.colptr, rowidx_out[:n], values_out[:n])


def ws_status(ws: torch.Tensor, stream=None) -> int:
    """Synchronizes and returns the device-side status of a workspace."""
    return int(_lib.spgemm_ws_status(_ptr(ws), _stream(stream)))


def ws_invalidate(ws: torch.Tensor, stream=None):
    """Drops what the workspace keeps between numeric calls (the slabbed copy of A)."""
    _check(_lib.spgemm_ws_invalidate(_ptr(ws), _stream(stream)), "spgemm_ws_invalidate")


def ws_status_code(ws: torch.Tensor, stream=None) -> tuple[int, int]:
    """(status, first device-side code) of a workspace; clears the code."""
    code = ctypes.c_int32(0)
    rc = int(_lib.spgemm_ws_status_code(_ptr(ws), _stream(stream), ctypes.byref(code)))
    return rc, int(code.value)


def check_ws(ws: torch.Tensor, where: str = "device check", stream=None):
    rc, code = ws_status_code(ws, stream)
    _check(rc, f"{where} (device code {code})" if code else where)


_lib.spgemm_ws_status_many.argtypes = [_vp, _i32, _vp, _vp]


def check_many(workspaces, where: str = "device check", stream=None):
    """check_ws for several workspaces with one synchronization; the first
    recorded code is raised."""
    n = len(workspaces)
    codes = (_i32 * n)()
    rc = int(_lib.spgemm_ws_status_many((_vp * n)(*[_ptr(w) for w in workspaces]), n, _stream(stream), codes))
    code = next((c for c in codes if c), 0)
    _check(rc, f"{where} (device code {code})" if code else where)


# -------------------------------------------------------------- batch loop
def layer_bounds(kdim: int, n_layers: int) -> list[tuple[int, int]]:
    """The inner-dimension ranges the library uses for n_layers layers."""
    w = -(-kdim // n_layers) if n_layers > 0 else kdim
    return [(min(kdim, l * w), min(kdim, l * w + w)) for l in range(n_layers)]


class _Unread:
    """Counts on the device, and the event after which they may be read (on
    any stream)."""

    def __init__(self, counts: torch.Tensor):
        self.counts = counts
        self.ready = torch.cuda.Event()
        self.ready.record()

    def read(self) -> np.ndarray:
        self.ready.synchronize()
        return self.counts.cpu().numpy()


@dataclass
class Plan:
    """Result of the symbolic pass and the planner for one product."""

    flops: torch.Tensor  # int64 [n] per output column (device)
    nnz: torch.Tensor  # int64 [rows, n] (device)
    nnz_host: np.ndarray  # int64 [rows, n]; read back on first use where the plan did not need it
    bounds: list
    batch_nnz: np.ndarray  # [b, rows]
    n_layers: int
    budget_bytes: int
    input_bytes: int
    reserve_bytes: int
    longest: int | None = None  # entries of C's longest column, if known
    row_longest: np.ndarray | None = None  # [rows] the same of every layer's product, and C's, if known

    @property
    def counts(self):
        """nnz_host, or where it has not been read back the tensor it comes from."""
        c = self.__dict__["nnz_host"]
        return c.counts if isinstance(c, _Unread) else c

    @property
    def nbatches(self) -> int:
        return len(self.bounds) - 1

    @property
    def total_flops(self) -> int:
        return int(self.flops.sum())

    def _read_counts(self) -> np.ndarray:
        c = self.__dict__["nnz_host"]
        if isinstance(c, _Unread):
            c = self.__dict__["nnz_host"] = c.read()
        return c

    def _set_counts(self, c):
        self.__dict__["nnz_host"] = c

    def __getstate__(self):  # saved or copied: with the counts themselves
        self._read_counts()
        return dict(self.__dict__)


# a field to the constructor, to dataclasses and to saved plans, read when asked for
Plan.nnz_host = property(Plan._read_counts, Plan._set_counts)


class Engine:
    """Holds workspaces and output buffers for repeated products of one shape.

    run(A, B) performs: symbolic pass -> counts to host -> batch planner ->
    per batch (numeric per layer [-> merge]) -> consume(c0, c1, C_batch).
    """

    def __init__(self, A, B, n_layers: int = 1, budget_bytes: int | None = None, max_batches: int = 1 << 16,
                 device="cuda", semiring=PLUS_TIMES, sorted_output: bool = False, esc_cf: float = ESC_CF_DEFAULT):
        if A.ncols != B.nrows:
            raise SpgemmError(E_SHAPE, "Engine")
        self.A, self.B, self.L = A, B, int(n_layers)
        self.semiring = semiring_id(semiring)
        # row-sorted output columns: each batch is formed, then sorted into a
        # second buffer of the same size (counted by the planner); with one
        # layer, columns of compression ratio up to esc_cf (and at most 4096
        # terms) are formed in row order directly (0: every column hashed)
        self.sorted_output = bool(sorted_output)
        self.esc_cf = float(esc_cf)
        self.device = device
        self.max_batches = max_batches
        self.vbytes = 4 if A.values is None or A.values.dtype == torch.float32 else 8
        self.vdtype = torch.float32 if self.vbytes == 4 else torch.float64
        n = B.ncols
        self.ws_sym = alloc_workspace(workspace_size(OP_SYMBOLIC, A, B, 0, n, self.L), device)
        self.ws_num = alloc_workspace(workspace_size(OP_NUMERIC, A, B, 0, n, self.L), device)
        mparts = CSC(A.nrows, n, A.colptr, A.rowidx, A.values)
        self.ws_mrg = alloc_workspace(workspace_size(OP_MERGE, mparts, None, 0, 0, max(1, self.L)), device) \
            if self.L > 1 else None
        # (the scan's status is not asked for: its header needs no clearing)
        self.ws_scan = torch.empty(workspace_size(OP_COLPTR, None, None, 0, n + 1), dtype=torch.uint8, device=device)
        self.ws_sort = alloc_workspace(workspace_size(OP_SORT, CSC(A.nrows, n, B.colptr, B.rowidx, B.values)), device) \
            if self.sorted_output and self.L > 1 else None
        rows = self.L + 1 if self.L > 1 else 1
        self.flops = torch.empty(n, dtype=torch.int64, device=device)
        self.nnz = torch.empty((rows, n), dtype=torch.int64, device=device)
        r = 4 + self.vbytes
        self.input_bytes = r * (A.nnz + B.nnz) + 8 * (A.ncols + B.ncols + 2)
        self.reserve_bytes = sum(int(w.numel()) for w in (self.ws_sym, self.ws_num, self.ws_mrg, self.ws_scan,
                                                          self.ws_sort) if w is not None) + 8 * 4 * (n + 1) * rows
        if budget_bytes is None:
            free, _ = torch.cuda.mem_get_info()
            budget_bytes = int(free * 0.9) + self.input_bytes + self.reserve_bytes
        self.budget_bytes = int(budget_bytes)
        self._bufs = {}  # output buffers of run_batch and staging of a whole product, by name

    # -- passes --------------------------------------------------------------
    def plan(self, stream=None) -> Plan:
        A, B, n = self.A, self.B, self.B.ncols
        # a product starts from scratch: its batches share one slabbed copy of A
        # (with few rows there is none)
        if A.nrows > SLAB_MIN_ROWS:
            ws_invalidate(self.ws_num, stream)
        symbolic(A, B, 0, n, self.L, self.flops, self.nnz, self.ws_sym, stream)
        whole = self._plan_whole(stream)
        if whole is not None:
            return whole
        with _on_stream(stream):  # where the symbolic pass is still at work
            nnz_host = self.nnz.cpu().numpy()
        counts = nnz_host
        if self.sorted_output:  # the merged batch is held twice: as formed and sorted
            counts = nnz_host.copy()
            counts[-1] *= 2
        bounds, tot = plan_batches(counts.reshape(-1), n, self.L, self.vbytes, self.input_bytes, self.budget_bytes,
                                   self.reserve_bytes, self.max_batches)
        if self.sorted_output:
            tot[:, -1] //= 2
        return Plan(self.flops, self.nnz, nnz_host, bounds, tot, self.L, self.budget_bytes, self.input_bytes,
                    self.reserve_bytes, int(nnz_host[-1].max(initial=0)), nnz_host.max(axis=1, initial=0))

    def _plan_whole(self, stream=None) -> Plan | None:
        """The plan of a product that fits as a whole, from sums formed on the
        device: reading the counts of 262,144 columns back and planning them on
        the host kept the GPU waiting for 1.0 ms.  None: the planner decides
        (and below 32,768 counts its way is the shorter)."""
        n, L = self.B.ncols, self.L
        rows = L + 1 if L > 1 else 1
        if n * rows < 32768 or rows > COUNT_SUMS_MAX_ROWS:
            return None
        sums = np.zeros(rows, np.int64)
        longest = np.zeros(rows, np.int64)
        _check(_lib.spgemm_count_sums_rows(_ptr(self.nnz), n, rows, sums.ctypes.data, longest.ctypes.data,
                                           _ptr(self.ws_scan), self.ws_scan.numel(), _stream(stream)),
               "spgemm_count_sums_rows")
        avail = self.budget_bytes - self.input_bytes - self.reserve_bytes
        held = int(sums[-1]) * (2 if self.sorted_output else 1) + (int(sums[:-1].sum()) if L > 1 else 0)
        if (4 + self.vbytes) * held + 8 * (L + 1 if L > 1 else 1) * n > avail or self.max_batches < 1:
            return None
        with _on_stream(stream):
            counts = _Unread(self.nnz.clone())  # self.nnz is written again by the next product
        return Plan(self.flops, self.nnz, counts, [0, n], sums.reshape(1, rows), L, self.budget_bytes,
                    self.input_bytes, self.reserve_bytes, int(longest[-1]), longest)

    def _hold(self, name: str, count: int, dtype) -> torch.Tensor:
        """The engine's buffer of that name, of at least ``count`` elements
        (the planner leaves room for one of each)."""
        t = self._bufs.get(name)
        if t is None or t.numel() < count:
            t = None
            self._bufs.pop(name, None)  # replaced, not joined
            t = self._bufs[name] = torch.empty(max(1, int(count)), dtype=dtype, device=self.device)
        return t

    def _hashed(self, plan: Plan):
        """(rows, values) of the largest batch, in hash-table order."""
        size = plan.batch_nnz[:, -1].max(initial=0)
        return self._hold("cri", size, torch.int32), self._hold("cv", size, self.vdtype)

    def _partials(self, plan: Plan):
        """(rows, values) of the partial products of the batch with most."""
        part = plan.batch_nnz[:, :self.L].sum(1).max(initial=0)
        return self._hold("dri", part, torch.int32), self._hold("dv", part, self.vdtype)

    def release_buffers(self):
        """Drops the output buffers (they are allocated again, at the size the next plan needs)."""
        self._bufs = {}

    def run_batch(self, plan: Plan, i: int, stream=None, marks=None) -> CSC:
        """Forms batch i; the returned CSC views buffers reused by the next call.
        With ``marks`` (a list), (phase, start_event, end_event) tuples are
        appended for the numeric and merge phases (HIP events on the stream)."""
        A, B, L = self.A, self.B, self.L

        def mark():
            if marks is None:
                return None
            e = torch.cuda.Event(enable_timing=True)
            e.record(stream if isinstance(stream, torch.cuda.Stream) else torch.cuda.current_stream())
            return e
        c0, c1 = plan.bounds[i], plan.bounds[i + 1]
        w = c1 - c0
        wmax = max(b - a for a, b in zip(plan.bounds[:-1], plan.bounds[1:]))
        ccp = self._hold("ccp", wmax + 1, torch.int64)[:w + 1]
        hashed = self._hashed(plan)
        nnzc = int(plan.batch_nnz[i, -1])
        out = hashed
        if self.sorted_output:
            size = plan.batch_nnz[:, -1].max()
            out = self._hold("sri", size, torch.int32), self._hold("sv", size, self.vdtype)
        parts = []
        e0 = mark()
        if L > 1:
            held = self._hold("dcp", L * (wmax + 1), torch.int64)
            dri, dv = self._partials(plan)
            off = 0
            for l in range(L):
                dcp = held[l * (w + 1):(l + 1) * (w + 1)]
                colptr(self.nnz[l, c0:c1], dcp, self.ws_scan, stream)
                cnt = int(plan.batch_nnz[i, l])
                parts.append(CSC(A.nrows, w, dcp, dri[off:off + cnt], dv[off:off + cnt]))
                off += cnt
        colptr(self.nnz[L if L > 1 else 0, c0:c1], ccp, self.ws_scan, stream)
        self._form(plan, i, ccp, nnzc, parts, hashed, out, stream, mark, e0, marks)
        return CSC(A.nrows, w, ccp, out[0][:nnzc], out[1][:nnzc])

    def _form(self, plan: Plan, i: int, ccp, nnzc: int, parts, hashed, out, stream=None, mark=lambda: None, e0=None,
              marks=None):
        """Batch i at the positions of the column pointers ccp: into ``out``
        (rows, values), with ``hashed`` holding the unsorted columns of a
        row-sorted product and ``parts`` the partial products of a layered one
        (tensors, or addresses that the pointers count from)."""
        A, B, L = self.A, self.B, self.L
        c0, c1 = plan.bounds[i], plan.bounds[i + 1]
        top = NO_BOUND if plan.longest is None else plan.longest
        if L == 1:
            if self.sorted_output:  # formed in row order (hashed columns staged)
                numeric_sorted(A, B, c0, c1, self.flops[c0:c1], ccp, *out, *hashed, self.ws_num, stream,
                               self.semiring, self.esc_cf, top)
            else:
                numeric(A, B, c0, c1, 0, 1, self.flops[c0:c1], ccp, *out, self.ws_num, stream, self.semiring, top)
            if marks is not None:
                marks.append(("numeric_sorted" if self.sorted_output else "numeric", e0, mark()))
            return
        for l, D in enumerate(parts):
            # the layer's own bound: C may have columns that need the slabbed copy
            # of A where none of the layer's does
            numeric(A, B, c0, c1, l, L, self.flops[c0:c1], D.colptr, D.rowidx, D.values, self.ws_num, stream,
                    self.semiring, top if plan.row_longest is None else int(plan.row_longest[l]))
        e1 = mark()
        merge(parts, ccp, *hashed, self.ws_mrg, stream, self.semiring)
        e2 = mark()
        if self.sorted_output:
            Cu = spgemm_csc(int(A.nrows), c1 - c0, nnzc, _ptr(ccp), _ptr(hashed[0]), _ptr(hashed[1]),
                            _DTYPE[self.vdtype])
            _check(_lib.spgemm_sort_columns(ctypes.byref(Cu), _ptr(out[0]), _ptr(out[1]), _ptr(self.ws_sort),
                                            self.ws_sort.numel(), _stream(stream)), "spgemm_sort_columns")
        if marks is not None:
            marks.append(("numeric", e0, e1))
            marks.append(("merge", e1, e2))
            if self.sorted_output:
                marks.append(("sort", e2, mark()))

    def _whole(self, plan: Plan, stream=None) -> CSC:
        """Every batch formed at its place in one output: nothing is copied, and
        one scan gives the column pointers of all batches (of all layers).
        1.3e9 bytes of rows and as many of values took 2.4 ms to copy twice."""
        A, L, n = self.A, self.L, self.B.ncols
        dev = self.device
        sizes = plan.batch_nnz[:, -1]
        total = int(sizes.sum())
        cp = torch.empty(n + 1, dtype=torch.int64, device=dev)
        ri = torch.empty(max(1, total), dtype=torch.int32, device=dev)
        v = torch.empty(max(1, total), dtype=self.vdtype, device=dev)
        vb = self.vbytes
        staged = self._hashed(plan) if self.sorted_output else None
        if L > 1:
            dri, dv = self._partials(plan)
            dcp = self._hold("dcp", L * n + 1, torch.int64)
            ws = self._hold("wcp", workspace_size(OP_COLPTR, None, None, 0, L * n), torch.uint8)
        # the memory comes from the current stream's pool, where what held it
        # before may still be at work (run() waits for ``stream`` before it
        # hands the output on)
        _wait_for_current(stream)
        colptr(self.nnz[L if L > 1 else 0], cp, self.ws_scan, stream)
        if L > 1:  # the layers' counts one after another: layer l's pointers start at l * n
            colptr(self.nnz[:L].reshape(-1), dcp, ws, stream)
            before = np.concatenate([[0], np.cumsum(plan.batch_nnz[:, :L].sum(0))])  # entries of earlier layers
        off = 0
        done = np.zeros(max(1, L), np.int64)
        for i in range(plan.nbatches):
            c0, c1 = plan.bounds[i], plan.bounds[i + 1]
            parts = []
            if L > 1:
                at = 0
                for l in range(L):
                    s = int(before[l] + done[l])  # the pointers' count at this batch's first column
                    cnt = int(plan.batch_nnz[i, l])
                    parts.append(spgemm_csc(int(A.nrows), c1 - c0, cnt, _ptr(dcp) + 8 * (l * n + c0),
                                            _ptr(dri) + 4 * (at - s), _ptr(dv) + vb * (at - s),
                                            _DTYPE[self.vdtype]))
                    at += cnt
                done += plan.batch_nnz[i, :L]
            out = (_ptr(ri), _ptr(v))
            hashed = (_ptr(staged[0]) - 4 * off, _ptr(staged[1]) - vb * off) if self.sorted_output else out
            self._form(plan, i, cp[c0:c1 + 1], int(sizes[i]), parts, hashed, out, stream)
            off += int(sizes[i])
        return CSC(A.nrows, n, cp, ri[:total], v[:total])

    def check(self, stream=None):
        check_many([w for w in (self.ws_sym, self.ws_num, self.ws_mrg, self.ws_sort) if w is not None],
                   "device-side check", stream)

    def run(self, consume=None, stream=None):
        """All batches; consume(c0, c1, C_batch) per batch, or the whole C."""
        stream = _stream(stream)  # looked up once
        plan = self.plan(stream)
        if consume is None:
            C = self._whole(plan, stream)
            self.check(stream)
            return C, plan
        for i in range(plan.nbatches):
            consume(plan.bounds[i], plan.bounds[i + 1], self.run_batch(plan, i, stream))
        self.check(stream)
        return plan


def _concat(batches, nrows):
    ncols = sum(b.ncols for b in batches)
    cps = []
    off = 0
    for b in batches:
        cps.append(b.colptr[:-1] + off)
        off += b.nnz
    dev = batches[0].rowidx.device if batches else "cuda"
    cps.append(torch.tensor([off], dtype=torch.int64, device=dev))
    return CSC(nrows, ncols, torch.cat(cps), torch.cat([b.rowidx for b in batches]),
               torch.cat([b.values for b in batches]))


def spgemm(A, B, *, layers: int = 1, budget_bytes: int | None = None, consume=None, stream=None,
           semiring=PLUS_TIMES, sorted_output: bool = False, esc_cf: float = ESC_CF_DEFAULT):
    """C = A B over ``semiring`` ('plus_times', 'min_plus', 'or_and'), rows of
    each column in hash-table order or, with ``sorted_output``, ascending.
    With ``consume`` the batches are handed to it and discarded; otherwise C
    is returned (all batches concatenated)."""
    eng = Engine(A, B, layers, budget_bytes, semiring=semiring, sorted_output=sorted_output, esc_cf=esc_cf)
    res = eng.run(consume, stream)
    return res if consume is not None else res[0]


# ------------------------------------------------------ consumer of a batch
_lib.spgemm_prune_topk.argtypes = [_P, ctypes.c_double, _i64, _vp, _vp, _vp, _i64, _vp, _sz, _vp]


def prune_bound(nnz: int, ncols: int, k: int) -> int:
    """Most entries a pruned matrix can hold: min(nnz, k * ncols), nnz for k < 0."""
    return nnz if k < 0 else min(nnz, k * ncols)


def prune_topk(C, threshold: float, k: int, ws: torch.Tensor | None = None, stream=None) -> CSC:
    """Per-column pruning of an output batch (the consumer an application
    runs on each batch): entries >= threshold, then at most the k largest of
    each column (k < 0: no limit), equal values going to the smaller row;
    kept entries stay in input order.  Reads the entry count back to the
    host and checks the workspace status."""
    if C.values is None:
        raise ValueError("prune_topk needs values")
    dev = C.rowidx.device
    if ws is None:
        ws = alloc_workspace(workspace_size(OP_PRUNE, C), dev)
    cap = prune_bound(C.nnz, C.ncols, int(k))
    cp = torch.empty(C.ncols + 1, dtype=torch.int64, device=dev)
    ri = torch.empty(max(1, cap), dtype=torch.int32, device=dev)
    v = torch.empty(max(1, cap), dtype=C.values.dtype, device=dev)
    _check(_lib.spgemm_prune_topk(ctypes.byref(desc(C)), float(threshold), int(k), _ptr(cp), _ptr(ri), _ptr(v), cap,
                                  _ptr(ws), ws.numel(), _stream(stream)), "spgemm_prune_topk")
    check_ws(ws, "device-side check (prune)", stream)
    n = int(cp[-1])
    return CSC(C.nrows, C.ncols, cp, ri[:n], v[:n])


def spgemm_topk(A, B, threshold: float, k: int, *, layers: int = 1, budget_bytes: int | None = None,
                stream=None) -> CSC:
    """C = A B formed batch by batch, every batch pruned as it is formed
    (``prune_topk``: entries >= threshold, at most the k largest per column)
    and only the pruned batches kept, concatenated: the whole product never
    needs to fit in memory, only one batch of it."""
    eng = Engine(A, B, layers, budget_bytes)
    ws = {}
    kept = []

    def consume(c0, c1, Cb):
        need = workspace_size(OP_PRUNE, Cb)
        if "ws" not in ws or ws["ws"].numel() < need:
            ws["ws"] = alloc_workspace(need, Cb.rowidx.device)
        kept.append(prune_topk(Cb, threshold, k, ws=ws["ws"], stream=stream))

    eng.run(consume, stream)
    if not kept:  # no batches
        dev = A.rowidx.device
        return CSC(A.nrows, B.ncols, torch.zeros(B.ncols + 1, dtype=torch.int64, device=dev),
                   torch.zeros(0, dtype=torch.int32, device=dev), torch.zeros(0, dtype=A.values.dtype, device=dev))
    return _concat(kept, A.nrows)


# ------------------------------------------------------------ gradient support
_lib.spgemm_transpose.argtypes = [_P, _vp, _vp, _vp, _vp, _vp, _sz, _vp]
_lib.spgemm_longest_row.argtypes = [_P, ctypes.POINTER(_i64), _vp, _sz, _vp]
_lib.spgemm_masked_xty.argtypes = [_P, _P, _P, _vp, _vp, _sz, _vp]
_lib.spgemm_permute.argtypes = [_vp, _vp, _i64, _i32, _i32, _vp, _vp]


def transpose(X, ws: torch.Tensor | None = None, values: bool = True, perm: bool = True, stream=None):
    """X^T as a CSC (values optional) and the permutation perm with
    X^T.values[q] = X.values[perm[q]]."""
    dev = X.rowidx.device
    if ws is None:
        ws = alloc_workspace(workspace_size(OP_TRANSPOSE, X), dev)
    tcp = torch.empty(X.nrows + 1, dtype=torch.int64, device=dev)
    tri = torch.empty(max(1, X.nnz), dtype=torch.int32, device=dev)
    tv = torch.empty(max(1, X.nnz), dtype=X.values.dtype, device=dev) if (values and X.values is not None) else None
    pm = torch.empty(max(1, X.nnz), dtype=torch.int64, device=dev) if perm else None
    _check(_lib.spgemm_transpose(ctypes.byref(desc(X)), _ptr(tcp), _ptr(tri), _ptr(tv), _ptr(pm), _ptr(ws),
                                 ws.numel(), _stream(stream)), "spgemm_transpose")
    n = X.nnz
    T = CSC(X.ncols, X.nrows, tcp, tri[:n], None if tv is None else tv[:n])
    return T, (None if pm is None else pm[:n])


def masked_xty(X, Y, M, out: torch.Tensor | None = None, ws: torch.Tensor | None = None, stream=None):
    """out(k,j) = sum_i X(i,k) Y(i,j) for each stored (k,j) of M, in M's order."""
    dev = Y.rowidx.device
    if ws is None:
        ws = alloc_workspace(workspace_size(OP_MASKED_XTY, X, Y, 0, Y.ncols), dev)
    if out is None:
        out = torch.empty(max(1, M.nnz), dtype=Y.values.dtype, device=dev)
    Md = desc(M, F32)
    Md.values = None
    _check(_lib.spgemm_masked_xty(ctypes.byref(desc(X)), ctypes.byref(desc(Y)), ctypes.byref(Md), _ptr(out), _ptr(ws),
                                  ws.numel(), _stream(stream)), "spgemm_masked_xty")
    return out[:M.nnz]


def permute(src: torch.Tensor, perm: torch.Tensor, scatter: bool = False, out: torch.Tensor | None = None,
            stream=None) -> torch.Tensor:
    """Gather out[i] = src[perm[i]] or scatter out[perm[i]] = src[i]."""
    n = perm.numel()
    if out is None:
        out = torch.empty(n, dtype=src.dtype, device=src.device)
    _check(_lib.spgemm_permute(_ptr(src), _ptr(perm), n, _DTYPE[src.dtype], int(scatter), _ptr(out), _stream(stream)),
           "spgemm_permute")
    return out


# Largest column of C whose gradient terms the fused backward forms (the
# largest LDS table is at most half full).
FUSED_COL_MAX = 5120
# Longest row of B, and entries of C (or B) per entry of it, from which the
# adds to one address bound the fused backward: each takes about 12 ns (22 where
# A's column is long), whatever else there is to do.  Called again and again, by
# float32 (float64 likewise), n = 262,144, a row of B in every column: 3.20 ms
# against 1.77 by transposed patterns at 1 entry of C per entry of the row,
# 3.22 against 2.85 at 64, 5.81 against 3.89 at 128 (columns of A of 32), but
# 6.5 against 20.2 at 509; a row in a quarter of 1e6 columns: 3.56 against 3.80
# at 64.  Rows of 4096: 77 against 88 us; of 8192: 126 against 122-130.
HUB_ROW_MIN = 4096
HUB_ROW_TERMS = 128


def _hub_row(longest_row: int, nnz_b: int, nnz_c: int) -> bool:
    """Whether adds to the same entries of dA would bound the fused backward
    (it has about as many terms as B or C has entries, or more)."""
    return longest_row > HUB_ROW_MIN and max(nnz_b, nnz_c) < HUB_ROW_TERMS * longest_row


def _longest_row(M, stream=None) -> int:
    """Entries of M's longest row."""
    out = _i64(0)
    ws = alloc_workspace(workspace_size(OP_TRANSPOSE, M), M.rowidx.device)
    _wait_for_current(stream)
    _check(_lib.spgemm_longest_row(ctypes.byref(desc(M)), ctypes.byref(out), _ptr(ws), ws.numel(), _stream(stream)),
           "spgemm_longest_row")
    return int(out.value)


def _fused_backward(A, B, b_values, C, dC_values, ws, stream=None):
    """dA and dB in one traversal of the product's terms (no transposes);
    every column of C must hold at most FUSED_COL_MAX entries."""
    if dC_values.dtype != A.values.dtype or b_values.dtype != A.values.dtype:
        raise SpgemmError(E_DTYPE, "spgemm_batched_backward")
    dev = C.rowidx.device
    dA = torch.empty(max(1, A.nnz), dtype=dC_values.dtype, device=dev)
    dB = torch.empty(max(1, B.nnz), dtype=dC_values.dtype, device=dev)
    bd = desc(CSC(B.nrows, B.ncols, B.colptr, B.rowidx, b_values))
    cd = desc(CSC(C.nrows, C.ncols, C.colptr, C.rowidx, None), F32)
    _check(_lib.spgemm_batched_backward(ctypes.byref(desc(A)), ctypes.byref(bd), ctypes.byref(cd), _ptr(dC_values),
                                        _ptr(dA), _ptr(dB), _ptr(ws), ws.numel(), _stream(stream)),
           "spgemm_batched_backward")
    return dA[:A.nnz], dB[:B.nnz]


def _on_stream(stream):
    """Context in which torch's own work goes to ``stream``: a torch stream or
    a handle (0: the default stream), or None for the current one."""
    if stream is None:
        return contextlib.nullcontext()
    if not isinstance(stream, torch.cuda.Stream):
        handle = _stream(stream)
        if handle == int(torch.cuda.current_stream().cuda_stream):
            return contextlib.nullcontext()
        # (an ExternalStream of handle 0 is not the default stream but another one)
        stream = torch.cuda.ExternalStream(handle) if handle else torch.cuda.default_stream()
    return torch.cuda.stream(stream)


def _wait_for_current(stream):
    """Work queued on ``stream`` from here on waits for the current stream's."""
    if stream is None:
        return
    current = torch.cuda.current_stream()
    if _stream(stream) != int(current.cuda_stream):
        with _on_stream(stream):
            torch.cuda.current_stream().wait_stream(current)


class Backward:
    """Gradients of a loss on P(C), C = A B, with respect to the stored values
    of A and B (B's as they were here or at the last refresh_values).

    Where no column of C holds more than FUSED_COL_MAX entries, both come from
    one traversal of the product's terms: 16.8e6 terms in float64 take 0.25 ms,
    against 0.92 ms by two masked products and two permutations over patterns
    already transposed (0.33 against 0.57 ms on a scale 12 R-MAT graph, whose
    hubs many columns add to at once).  Longer columns have no LDS table to
    hold them, and a row of B with most of the entries (see HUB_ROW_MIN) makes
    the traversal wait for the adds to a few entries of dA: then the transposes
    of A's and B's patterns and of C's pattern are formed once (per structure)
    and reused."""

    _LAZY = ("ws_tr", "AT", "permA", "CT", "permC", "BT", "permB", "ws_b", "ws_a")

    def __init__(self, A, B, C, stream=None):
        self.A, self.B, self.C = A, B, C
        self.ws_f = None
        with _on_stream(stream):
            longest = int((C.colptr[1:] - C.colptr[:-1]).max()) if C.ncols > 0 else 0
        fused = longest <= FUSED_COL_MAX and A.values is not None and B.values is not None
        if fused and _hub_row(B.ncols, B.nnz, C.nnz):  # (a row holds at most one entry per column)
            fused = not _hub_row(_longest_row(B, stream), B.nnz, C.nnz)
        if fused:
            # both from the current stream's pool, as all memory here: gradients
            # may be asked for on another stream than this one
            self._b = torch.empty_like(B.values)
            self.ws_f = alloc_workspace(workspace_size(OP_BATCHED_BACKWARD, A, B, 0, C.ncols), C.rowidx.device)
            _wait_for_current(stream)
            with _on_stream(stream):
                self._b.copy_(B.values.detach())
        if self.ws_f is None:
            self._transposes(B, stream)

    def _transposes(self, B, stream=None):
        A, C = self.A, self.C
        dev = C.rowidx.device
        self.ws_tr = alloc_workspace(max(workspace_size(OP_TRANSPOSE, M) for M in (A, B, C)), dev)
        self.AT, self.permA = transpose(A, self.ws_tr, values=False, perm=True, stream=stream)
        self.CT, self.permC = transpose(C, self.ws_tr, values=False, perm=True, stream=stream)
        self.BT, self.permB = transpose(B, self.ws_tr, values=True, perm=True, stream=stream)
        self.ws_b = alloc_workspace(workspace_size(OP_MASKED_XTY, A, C, 0, C.ncols), dev)
        self.ws_a = alloc_workspace(workspace_size(OP_MASKED_XTY, self.BT, self.CT, 0, self.CT.ncols), dev)

    def __getattr__(self, name):
        # the fused form makes the transposed patterns only when asked for them
        if name in Backward._LAZY and self.__dict__.get("ws_f") is not None:
            B = self.B
            self._transposes(CSC(B.nrows, B.ncols, B.colptr, B.rowidx, self._b))
            return self.__dict__[name]
        raise AttributeError(name)

    def refresh_values(self, B, stream=None):
        """New values of B (same pattern)."""
        self.B = B
        if self.ws_f is not None:
            with _on_stream(stream):
                self._b.copy_(B.values.detach())  # not a step of any graph
        if "BT" in self.__dict__:  # B^T's values are re-gathered
            permute(B.values, self.permB, False, self.BT.values, stream)

    def __call__(self, dC_values: torch.Tensor, stream=None):
        A, B, C = self.A, self.B, self.C
        if self.ws_f is not None:
            return _fused_backward(A, B, self._b, C, dC_values, self.ws_f, stream)
        Y = CSC(C.nrows, C.ncols, C.colptr, C.rowidx, dC_values)
        dB = masked_xty(A, Y, B, ws=self.ws_b, stream=stream)
        dCT = permute(dC_values, self.permC, False, stream=stream)
        YT = CSC(self.CT.nrows, self.CT.ncols, self.CT.colptr, self.CT.rowidx, dCT)
        dAT = masked_xty(self.BT, YT, self.AT, ws=self.ws_a, stream=stream)
        dA = permute(dAT, self.permA, True, stream=stream)
        return dA, dB

    def check(self, stream=None):
        for w in (self.ws_f,) + tuple(self.__dict__.get(k) for k in ("ws_tr", "ws_b", "ws_a")):
            if w is not None:
                check_ws(w, "device-side check (backward)", stream)


class SpGEMMFn(torch.autograd.Function):
    """C.values = (A B).values as a function of A's and B's stored values;
    C's pattern (colptr, rowidx) is returned as non-differentiable outputs.

        c_vals, c_colptr, c_rowidx = SpGEMMFn.apply(a_vals, b_vals, A, B)

    A and B give the patterns (their own values are ignored)."""

    @staticmethod
    def forward(ctx, a_vals, b_vals, A, B, layers=1, budget_bytes=None):
        Av = CSC(A.nrows, A.ncols, A.colptr, A.rowidx, a_vals)
        Bv = CSC(B.nrows, B.ncols, B.colptr, B.rowidx, b_vals)
        C, plan = Engine(Av, Bv, layers, budget_bytes).run()
        ctx.longest = plan.longest
        ctx.set_materialize_grads(False)  # the pattern outputs need no gradients of zeros
        ctx.save_for_backward(a_vals, b_vals)
        ctx.A, ctx.B, ctx.C = A, B, CSC(C.nrows, C.ncols, C.colptr, C.rowidx, None)
        ctx.mark_non_differentiable(C.colptr, C.rowidx)
        return C.values, C.colptr, C.rowidx

    @staticmethod
    def backward(ctx, d_vals, _d_cp, _d_ri):
        a_vals, b_vals = ctx.saved_tensors
        if d_vals is None:  # a gradient of zeros
            return torch.zeros_like(a_vals), torch.zeros_like(b_vals), None, None, None, None
        A = CSC(ctx.A.nrows, ctx.A.ncols, ctx.A.colptr, ctx.A.rowidx, a_vals)
        B = CSC(ctx.B.nrows, ctx.B.ncols, ctx.B.colptr, ctx.B.rowidx, b_vals)
        # no transposes: see Backward (formed here, on every call, they cost more
        # than any row's adds: 8.6 ms against 3.3 in the worst case above)
        if ctx.longest <= FUSED_COL_MAX:
            ws = alloc_workspace(workspace_size(OP_BATCHED_BACKWARD, A, B, 0, B.ncols), ctx.C.rowidx.device)
            dA, dB = _fused_backward(A, B, b_vals, ctx.C, d_vals.contiguous(), ws)
            check_ws(ws, "device-side check (backward)")
        else:
            bw = Backward(A, B, ctx.C)
            dA, dB = bw(d_vals.contiguous())
            bw.check()
        return dA, dB, None, None, None, None
