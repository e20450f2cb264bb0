"""GPU parity at the row counts where a kernel changes its LDS structure:
the item kernel cuts its work queue into smaller batches when a product has
few heavy columns."""
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
