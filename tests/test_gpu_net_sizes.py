"""The network's kernels at the edges of their tiles (16 nodes per wave, 64
nodes per step and 2048 per chunk of the weight gradients, 16384 nodes where
the layer update changes its form) and on rows that are empty or long,
against the FP64 reference with the GPU's BF16 activation storage.  Bars as in
test_gpu_gnn.py: 1e-2 for predictions and the loss, 2e-2 per gradient block
(BF16 keeps 8 mantissa bits; a value rounds differently only where FP32 and
FP64 sums straddle a rounding boundary)."""
import numpy as np
import pytest
import scipy.sparse as sp

import lpgen
from tests.test_gpu_gnn import D, bf16_bits, bf16_value  # noqa: F401
from tests.test_gpu_tiles import ragged_lp

pytestmark = pytest.mark.gpu


def _lp(m, n, shape):
    if shape == "ragged":
        return ragged_lp(20, m, m, n)
    return lpgen.constructed_lp(m, n, m // 2, 4, seed=m + n)


@pytest.mark.parametrize("m,n,shape", [
    (5, 16, "uniform"), (17, 33, "uniform"), (63, 65, "uniform"), (700, 515, "ragged"),
    (2049, 4096, "uniform"), (2048, 2047, "uniform"), (16383, 16385, "uniform"),
    (16400, 16384, "uniform")])
def test_network_sizes_match_fp64_reference(D, m, n, shape):  # noqa: F811
    import oracle
    from oracle import gnn_ref
    from paper_2601_07628_amd import warmstart as W
    layers = 2
    lp = _lp(m, n, shape)
    rng = np.random.default_rng(m * n)
    p = W.init_params(layers, seed=m)
    p[-256:] = 0.05 * rng.standard_normal(256)
    x_ref, y_ref = rng.uniform(-1, 1, n), rng.standard_normal(m)
    tx, ty = x_ref + rng.standard_normal(n), y_ref + rng.standard_normal(m)
    b_ref = D.row_b(lp.con_lo, lp.con_hi)
    inst = lpgen.perturbed(lp, 9)
    net = D.WarmStartNet(D.Problem(lp), layers=layers)
    net.set_params(p)
    net.set_reference(lp.c, b_ref, x_ref, y_ref)
    net.set_instance(inst.c, inst.con_lo, inst.con_hi)
    x0, y0 = net.forward()
    loss = net.backward(tx, ty)
    _, g = net.params(grads=True)

    sd = oracle.Problem(lp, oracle.Params(eta=1.0, omega0=1.0)).scaled()
    dr, dc = sd["dr"], sd["dc"]
    A = sp.csr_matrix((sd["v"], lp.col_idx, lp.row_ptr), shape=(m, n))
    rnd = lambda v: bf16_value(bf16_bits(v)).reshape(v.shape)  # noqa: E731
    Xc, Xr = (rnd(v) for v in gnn_ref.features(inst.c, inst.con_lo, inst.con_hi, inst.var_lo,
                                               inst.var_hi, lp.c, b_ref, x_ref, y_ref, dr, dc))
    pq = p.astype(np.float64)
    pq[:-256] = rnd(p[:-256])
    px, py, _ = gnn_ref.forward(pq, layers, A, Xc, Xr, x_ref / dc, y_ref / dr, rnd)
    rel = lambda a, b: np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)  # noqa: E731
    assert rel(x0 / dc - x_ref / dc, px - x_ref / dc) < 1e-2
    assert rel(y0 / dr - y_ref / dr, py - y_ref / dr) < 1e-2
    L, gr = gnn_ref.loss_and_grad(pq, layers, A, Xc, Xr, x_ref / dc, y_ref / dr, tx / dc, ty / dr, rnd)
    assert abs(loss.sum() - L) <= 1e-2 * L
    d_g, d_r = gnn_ref.unpack(g, layers), gnn_ref.unpack(gr, layers)
    for name in ("W_cin", "W_rin", "w_x", "w_y"):
        assert rel(d_g[name], d_r[name]) < 2e-2, name
    for name in ("W_c", "W_r"):
        for l in range(layers):
            assert rel(d_g[name][l], d_r[name][l]) < 2e-2, (name, l)
