"""dpdlp_kkt_noalloc at the edges of its work split (32 rows or columns per
workgroup and round, 131072 per round of the whole launch, segments of more
than 64 entries taken by a whole wave) against App. B.4 evaluated with scipy
in FP64.  Bar: 1e-11 relative, as between the two GPU evaluations (sums of
up to 3e5 FP64 terms in another order differ by some 1e-14)."""
import numpy as np
import pytest
import scipy.sparse as sp

from tests.test_zz_no_alloc import D  # noqa: F401

pytestmark = pytest.mark.gpu


def _matrix(m, n, lens, rng):
    """Rows of the given lengths, distinct columns."""
    cols = np.concatenate([(rng.integers(n) + np.arange(d) * max(1, n // max(d, 1))) % n for d in lens])
    rows = np.repeat(np.arange(m), lens)
    key = np.unique(rows * n + cols)
    return sp.csr_matrix((rng.standard_normal(key.size), (key // n, key % n)), shape=(m, n))


@pytest.mark.parametrize("m,n,case", [
    (1, 1, "short"), (31, 33, "short"), (32, 64, "empty"), (500, 3000, "long rows"),
    (3000, 500, "long columns"), (131073, 40, "rounds"), (40, 131105, "rounds")])
@pytest.mark.parametrize("qp", [False, True])
def test_kkt_noalloc_sizes(D, m, n, case, qp):  # noqa: F811
    import torch
    rng = np.random.default_rng(m + n)
    lens = rng.integers(0 if case == "empty" else 1, min(n, 6) + 1, size=m)
    if case == "long rows":
        lens[[0, 7, 8, 499]] = [64, 65, 2999, 700]
    A = _matrix(m, n, lens, rng)
    if case == "long columns":
        A = sp.csr_matrix(_matrix(n, m, np.where(np.arange(n) % 9 == 0, 1500, 3), rng).T)
    x, y = rng.standard_normal(n), rng.standard_normal(m)
    c, dc = rng.standard_normal(n), rng.uniform(0.5, 2, n)
    clo = np.where(rng.random(m) < 0.3, -np.inf, rng.standard_normal(m))
    chi = np.where(rng.random(m) < 0.3, np.inf, np.where(np.isfinite(clo), clo, 0) + rng.random(m))
    y = np.where(np.isinf(chi), np.maximum(y, 0), y)
    y = np.where(np.isinf(clo), np.minimum(y, 0), y)
    vlo, vhi = np.full(n, -0.5), np.where(rng.random(n) < 0.5, np.inf, 0.7)
    q = rng.random(n) if qp else None
    tau = 0.37

    csr = dict(row_ptr=A.indptr, col_idx=A.indices, val=A.data, c=c, con_lo=clo, con_hi=chi,
               var_lo=vlo, var_hi=vhi)
    At = A.tocsc()
    csc = dict(col_ptr=At.indptr, row_idx=At.indices, val=At.data)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(  # noqa: E731
        v, np.int32 if np.issubdtype(np.asarray(v).dtype, np.integer) else np.float64)).cuda()
    out = torch.full((5,), np.nan, dtype=torch.float64, device="cuda")
    D.dpdlp_kkt_noalloc(m, n, {k: dev(v) for k, v in csr.items()}, {k: dev(v) for k, v in csc.items()},
                        dev(x), dev(y), tau, out, col_scale=dev(dc), q=None if q is None else dev(q),
                        stream=torch.cuda.current_stream())
    torch.cuda.synchronize()

    ax = A @ x
    qx = q * x if qp else np.zeros(n)
    g = c + qx - A.T @ y
    t = tau * dc * dc
    u = x - t * g
    s = (np.clip(u, vlo, vhi) - u) / t
    fin = np.concatenate([clo[np.isfinite(clo)], chi[np.isfinite(chi)]])
    py = np.sum(np.where(y > 0, clo, np.where(y < 0, chi, 0.0)) * np.where(y != 0, y, 1.0) * (y != 0))
    po, do = c @ x + qx @ x / 2, py + s @ x - qx @ x / 2
    want = [np.linalg.norm(ax - np.clip(ax, clo, chi)) / (1 + np.linalg.norm(fin)),
            np.linalg.norm(g - s) / (1 + np.linalg.norm(c)),
            abs(po - do) / (1 + max(abs(po), abs(do))), po, do]
    got = out.cpu().numpy()
    scale = np.array([1, 1, 1, 1 + abs(po), 1 + abs(do)])
    assert np.all(np.abs(got - want) <= 1e-11 * np.maximum(scale, np.abs(want))), (got, want)
