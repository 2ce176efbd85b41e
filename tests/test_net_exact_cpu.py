"""CPU checks of the exact network instances (net_exact.py): that every number
is held exactly, and that a mistake the size of one MFMA step, one chunk or one
node, planted in the reference, changes the result they are compared with."""
import numpy as np
import pytest

from oracle import gnn_ref
from tests import net_exact

H = net_exact.H


@pytest.mark.parametrize("m,n,layers,seed", net_exact.CASES)
def test_instances_are_exact(m, n, layers, seed):
    net_exact.check_exact(net_exact.instance(m, n, layers, seed))


@pytest.mark.parametrize("m,n,layers,seed", [(64, 63, 1, 1), (2049, 2048, 1, 1), (4096, 640, 1, 2)])
def test_planted_mistakes_show(m, n, layers, seed):
    I = net_exact.instance(m, n, layers, seed)
    A, At = I["A"], I["A"].T.tocsr()
    W = gnn_ref.unpack(I["p"], layers)
    px, py, c = gnn_ref.forward(I["p"], layers, A, *I["X"], I["ref"]["x"], I["ref"]["y"])
    dx, dy = 2 * (px - I["tx"]) / n, 2 * (py - I["ty"]) / m
    dZc = np.outer(dx, W["w_x"]) * (c["Hc"][0] > 0)
    gc = dZc @ W["W_c"][0].T
    dZr = (np.outer(dy, W["w_y"]) + A @ gc[:, H:]) * (c["Hr"][0] > 0)
    for IN, Wl, dZ in ((c["INc"][0], W["W_c"][0], dZc), (c["INr"][0], W["W_r"][0], dZr)):
        N = IN.shape[0]
        full = IN @ Wl
        for s in range(0, 2 * H, 16):           # a step of the layer update, at any node tile
            cut = full - IN[:, s:s + 16] @ Wl[s:s + 16]
            differs = (np.maximum(cut, 0) != np.maximum(full, 0)).any(axis=1)
            assert all(differs[t:t + 16].any() for t in range(0, N - N % 16, 16))
        for s in range(0, H, 16):               # a step of the data gradient
            assert (dZ[:, s:s + 16] @ Wl[:, s:s + 16].T).any()
        lo = dZ - net_exact.bf16(dZ)
        assert (IN.T @ lo).any()                # the low halves
        # the last node of each chunk and step of the weight gradient, and the first of the next
        for j in sorted({0, 1, N - 1, N - 2} | {e for q in range(2048, N, 2048) for e in (q - 1, q)}):
            assert np.outer(IN[j], dZ[j]).any(), j
    assert (At @ (dZr @ W["W_r"][0].T)[:, H:]).any()
