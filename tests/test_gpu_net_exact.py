"""The network's kernels (embedding, both forms of the layer update, sparse
products, heads, data and weight gradients) on instances in which every value
is held exactly: results equal the FP64 reference bit for bit, so a lost MFMA
step, a wrong lane or a node left out of a chunk fails."""
import numpy as np
import pytest

from oracle import gnn_ref
from tests import net_exact
from tests.test_gpu_gnn import D  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,layers,seed", net_exact.CASES)
def test_network_is_exact(D, m, n, layers, seed):  # noqa: F811
    I = net_exact.instance(m, n, layers, seed)
    lp, ref = I["lp"], I["ref"]
    net = D.WarmStartNet(D.Problem(lp, ruiz_iters=0, use_pc=0, eta=0.1), layers=layers)
    net.set_params(I["p"])
    net.set_reference(ref["c"], ref["b"], ref["x"], ref["y"])
    net.set_instance(lp.c, lp.con_lo, lp.con_hi)
    x0, y0 = net.forward()
    assert np.array_equal(x0, I["px"]) and np.array_equal(y0, I["py"])
    loss = net.backward(I["tx"], I["ty"])
    _, g = net.params(grads=True)
    L, gr = gnn_ref.loss_and_grad(I["p"], layers, I["A"], *I["X"], ref["x"], ref["y"], I["tx"], I["ty"])
    assert loss.sum() == L
    got, want = gnn_ref.unpack(g, layers), gnn_ref.unpack(gr, layers)
    for name in want:
        assert np.array_equal(got[name], want[name]), name
