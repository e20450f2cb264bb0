"""GPU parity at the row counts where a kernel changes its LDS structure:
the symbolic pass counts a column's rows in a bitmap instead of a hash table
up to 32 rows per slot of the bin's table, and the item kernel cuts its work
queue into smaller batches when a product has few heavy columns."""
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


def _csc(m, cols, dtype, rng):
    cp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    ri = np.concatenate(cols).astype(np.int32)
    return synth.CSC(m, len(cols), torch.from_numpy(cp), torch.from_numpy(ri),
                     torch.from_numpy(rng.standard_normal(ri.size)).to(dtype))


def _operands(m, seed, dtype=torch.float32):
    """A: columns of 1 to 200 rows that together touch the first and the last
    row of C; B: columns whose term counts fall into every bin."""
    rng = np.random.default_rng(seed)
    acols = [rng.choice(m, min(m, n), replace=False) for n in rng.integers(1, 200, 400)]
    acols += [np.unique([0, m - 1]), np.array([m - 1]), np.arange(max(0, m - 40), m), np.array([], np.int64)]
    k = len(acols)
    bcols = [np.array([], np.int64), np.array([k - 4]), np.array([k - 1]), np.array([k - 4, k - 3, k - 2, 0, 1])]
    for n in (1, 2, 3, 6, 12, 25, 60, 130, 250, k):
        bcols += [np.concatenate([rng.choice(k - 4, n - 1, replace=False), [k - 4]]) if n < k else np.arange(k)
                  for _ in range(3)]
    return _csc(m, acols, dtype, rng), _csc(k, bcols, dtype, rng)


@pytest.mark.parametrize("m", [1, 31, 33, 2047, 2048, 2049, 8192, 8193, 32768, 32769, 131072, 131073, 524289,
                               1048576, 1048577])
@pytest.mark.parametrize("layers", [1, 3])
def test_symbolic_counts_at_bitmap_limits(m, layers):
    print(f"case: bitmap limit m={m} layers={layers}", flush=True)
    A, B = _operands(m, 100 + m % 97)
    plan = S.Engine(A.to("cuda"), B.to("cuda"), layers).plan()
    assert np.array_equal(plan.nnz_host[-1], oracle.count(A, B))
    assert np.array_equal(plan.flops.cpu().numpy(), oracle.flops(A, B))
    if layers > 1:
        for l, (lo, hi) in enumerate(S.layer_bounds(A.ncols, layers)):
            assert np.array_equal(plan.nnz_host[l], oracle.count(A, B, klo=lo, khi=hi))


@pytest.mark.parametrize("heavy", [1, 5, 63, 64, 65, 300])
@pytest.mark.parametrize("m", [5200, 70000])
def test_item_batches_at_few_heavy_columns(heavy, m):
    """`heavy` columns of more than 5120 rows over 2 or 18 row slabs, one of
    them with more than 1024 entries of B."""
    print(f"case: item batches heavy={heavy} m={m}", flush=True)
    rng = np.random.default_rng(heavy)
    k = 1100
    A = _csc(m, [rng.choice(m, 60, replace=False) for _ in range(k)], torch.float64, rng)
    cols = [rng.choice(k, 1000 if m < 10000 else 200, replace=False) for _ in range(heavy)] + [np.arange(k)]
    cols += [rng.choice(k, 2, replace=False) for _ in range(7)]
    B = _csc(k, cols, torch.float64, rng)
    assert int((oracle.count(A, B) > 5120).sum()) == heavy + 1
    C, _ = S.Engine(A.to("cuda"), B.to("cuda")).run()
    assert_matches(C, oracle.spgemm(A, B), torch.float64, f"heavy={heavy} m={m}")


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 300])
def test_column_flops_and_counts(n):
    """Columns of B from empty to far longer than a wave's step, in groups
    that start and end with empty ones."""
    print(f"case: column flops n={n}", flush=True)
    rng = np.random.default_rng(n)
    k = 6000
    A = _csc(900, [rng.choice(900, c, replace=False) for c in rng.integers(0, 4, k)], torch.float64, rng)
    lens = rng.choice([0, 0, 1, 2, 63, 64, 65, 511, 512, 513, 5000], n)
    lens[-1] = 0
    lens[n // 2] = 1500
    B = _csc(k, [rng.choice(k, c, replace=False) for c in lens], torch.float64, rng)
    plan = S.Engine(A.to("cuda"), B.to("cuda")).plan()
    assert np.array_equal(plan.flops.cpu().numpy(), oracle.flops(A, B))
    assert np.array_equal(plan.nnz_host[0], oracle.count(A, B))


@pytest.mark.parametrize("n", [0, 1, 7, 8191, 8192, 8193, 100003, 8192 * 4096, 8192 * 4096 + 1])
def test_column_pointers(n):
    print(f"case: column pointers n={n}", flush=True)
    x = torch.randint(0, 1 << 33, (n + 1,), device="cuda", generator=torch.Generator("cuda").manual_seed(n))[1:]
    out = torch.full((n + 1,), -1, dtype=torch.int64, device="cuda")
    S.colptr(x, out, S.alloc_workspace(S.workspace_size(S.OP_COLPTR, None, None, 0, n)))
    assert int(out[0]) == 0 and torch.equal(out[1:], torch.cumsum(x, 0))
