"""Merged splits of 5 to 8 pieces against the CPU oracle, at sizes where the
merge rule takes each of its branches (64-nonzero tiles keep them small): left
as separate pieces, merged beside whole tiles, merged as many among many.  Bar:
the iterates' 1e-10 of the parity tests (another order of additions of rows of
up to 509 terms differs by some 1e-15)."""
import numpy as np
import pytest

import lpgen
from tests.test_gpu_parity import D, O, fixed_run  # noqa: F401

pytestmark = pytest.mark.gpu
TILE = 64


@pytest.mark.parametrize("rows,pieces,short", [
    (30, 5, 0), (6, 6, 300), (7, 5, 4000), (7, 6, 4000), (400, 5, 0), (40, 8, 4000), (70, 7, 42000),
    (70, 8, 42000)])
def test_merged_pieces_match_oracle(D, O, rows, pieces, short):  # noqa: F811
    rng = np.random.default_rng(rows + pieces + short)
    m, n = rows + short, 3000
    deg = rng.integers(1, 5, size=m)
    deg[rng.choice(m, size=rows, replace=False)] = pieces * TILE - 3
    cols = np.concatenate([np.sort(rng.choice(n, size=d, replace=False)) for d in deg])
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    val = rng.standard_normal(cols.size)
    x = rng.uniform(0, 1, n)
    ax = np.bincount(np.repeat(np.arange(m), deg), weights=val * x[cols], minlength=m)
    lp = lpgen.LP(m, n, rp, cols.astype(np.int32), val, rng.standard_normal(n), ax - 0.1,
                  np.full(m, np.inf), np.zeros(n), np.full(n, 2.0), name=f"merge{rows}x{pieces}")
    fixed_run(D, O, lp, 130, gpu_kw=dict(tile_nnz=TILE))
