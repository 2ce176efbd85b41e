"""The tile kernels at the edges of their instantiations: nonzeros per thread
(1, 2, 4, 8 by tile size) and every width of the segment reduction (1 to 64
lanes), against the CPU oracle.  Bar: the iterates' 1e-10 of the parity tests
(FP64 sums of up to 80 terms in another order differ by some 1e-15)."""
import numpy as np
import pytest

import lpgen
from tests.test_gpu_parity import D, O, fixed_run  # noqa: F401

pytestmark = pytest.mark.gpu


def ragged_lp(mean, seed, m=2311, n=1777):
    """Rows of 0 to 2 mean nonzeros, every seventh one empty, one free row."""
    rng = np.random.default_rng(seed)
    deg = rng.integers(0, 2 * mean + 1, size=m)
    deg[::7] = 0
    deg = np.minimum(deg, n)
    rows = np.repeat(np.arange(m), deg)
    cols = np.concatenate([np.sort(rng.choice(n, size=d, replace=False)) for d in deg])
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    val = rng.standard_normal(rows.size)
    x = rng.uniform(-1, 1, n)
    ax = np.bincount(rows, weights=val * x[cols], minlength=m)
    lo = np.where(rng.random(m) < 0.5, ax, ax - 0.5)
    hi = np.where(rng.random(m) < 0.5, np.maximum(lo, ax), np.inf)
    lo[3], hi[3] = -np.inf, np.inf
    return lpgen.LP(m, n, rp, cols.astype(np.int32), val, rng.standard_normal(n), lo, hi,
                    np.full(n, -1.0), np.full(n, 1.0), name=f"ragged{mean}")


@pytest.mark.parametrize("tile_nnz", [96, 256, 257, 512, 513, 1024, 1025, 2048])
def test_tile_sizes_around_the_instantiations(D, O, tile_nnz):  # noqa: F811
    fixed_run(D, O, ragged_lp(6, tile_nnz), 130, gpu_kw=dict(tile_nnz=tile_nnz))


@pytest.mark.parametrize("mean", [1, 2, 4, 8, 16, 40])
def test_segment_reduction_widths(D, O, mean):  # noqa: F811
    fixed_run(D, O, ragged_lp(mean, 50 + mean), 130)


@pytest.mark.parametrize("long_len", [65, 700, 2040])
def test_long_segments_among_short_ones(D, O, long_len):  # noqa: F811
    """Tiles that mix rows of 1 to 3 nonzeros with long rows (the summing
    width is chosen from the longest lanes of the tile's waves)."""
    rng = np.random.default_rng(long_len)
    m, n = 1500, 2100
    deg = rng.integers(1, 4, size=m)
    deg[rng.choice(m, size=9, replace=False)] = long_len
    cols = np.concatenate([np.sort(rng.choice(n, size=d, replace=False)) for d in deg])
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    val = rng.standard_normal(cols.size)
    x = rng.uniform(0, 1, n)
    ax = np.bincount(np.repeat(np.arange(m), deg), weights=val * x[cols], minlength=m)
    lp = lpgen.LP(m, n, rp, cols.astype(np.int32), val, rng.standard_normal(n), ax - 0.1,
                  np.full(m, np.inf), np.zeros(n), np.full(n, 2.0), name=f"long{long_len}")
    fixed_run(D, O, lp, 130, gpu_kw=dict(tile_nnz=2048))


@pytest.mark.parametrize("slices", [0, 8])
@pytest.mark.parametrize("pieces", [1, 2, 4, 5, 12])
def test_split_segments_merged_and_not(D, O, pieces, slices):  # noqa: F811
    """Rows of `pieces` tiles among short ones: up to eight pieces stay in one
    workgroup, more are added up by a launch of their own (unsliced) or by the
    combine (sliced); with rows of both kinds in one matrix."""
    rng = np.random.default_rng(10 * pieces + slices)
    m, n, tile = 900, 4000, 256
    deg = rng.integers(1, 6, size=m)
    deg[rng.choice(m, size=7, replace=False)] = pieces * tile - 3
    deg[rng.choice(m, size=2, replace=False)] = 3 * tile + 1
    deg[rng.choice(m, size=2, replace=False)] = 9 * tile
    cols = np.concatenate([np.sort(rng.choice(n, size=d, replace=False)) for d in deg])
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int32)
    val = rng.standard_normal(cols.size)
    x = rng.uniform(0, 1, n)
    ax = np.bincount(np.repeat(np.arange(m), deg), weights=val * x[cols], minlength=m)
    lp = lpgen.LP(m, n, rp, cols.astype(np.int32), val, rng.standard_normal(n), ax - 0.1,
                  np.full(m, np.inf), np.zeros(n), np.full(n, 2.0), name=f"pieces{pieces}")
    fixed_run(D, O, lp, 130, gpu_kw=dict(tile_nnz=tile, gather_slices=slices))
