"""Instances of the warm-start network whose every number is an integer that
BF16, a BF16 pair or FP32 holds exactly, so that the GPU's result must equal
the FP64 reference bit for bit, in whatever order it adds.

A has entries +-1 and is not rescaled; weights are +-1 on a few entries per
column, spread over all rows; the heads hold integers of up to 9 bits, so the
gradients need both BF16 halves.  Targets lie k N from the prediction (k in
{-1, 0, 1}), which makes the loss gradient 2 k.  check_exact() proves for an
instance that activations fit BF16, gradients a BF16 pair, and the sums of
absolute values 24 bits."""
import numpy as np
import scipy.sparse as sp

import lpgen
from oracle import gnn_ref

H, F = gnn_ref.H, gnn_ref.F


def bf16(v):
    """v rounded to BF16 (nearest even), as FP64."""
    u = np.ascontiguousarray(v, np.float32).view(np.uint32).astype(np.uint64)
    u = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16).astype(np.uint32) << 16
    return u.view(np.float32).astype(np.float64)


def _graph(m, n, most, rng):
    """+-1 entries: 0 to `most` per row, a few rows and columns of 9 to 41."""
    deg = rng.integers(0, most + 1, m)
    deg[::7] = 0
    for d in (9, 17, 41)[:most]:
        deg[rng.integers(m)] = d
    deg = np.minimum(deg, n)
    rows = np.repeat(np.arange(m), deg)
    cols = np.concatenate([rng.choice(n, d, replace=False) for d in deg] + [np.zeros(0, int)])
    for d in (16, 25)[:most]:
        d = min(d, m)
        rows = np.concatenate([rows, rng.choice(m, d, replace=False)])
        cols = np.concatenate([cols, np.full(d, rng.integers(n))])
    key = np.unique(rows * n + cols)
    val = rng.choice([-1.0, 1.0], key.size)
    return sp.csr_matrix((val, (key // n, key % n)), shape=(m, n))


def _weights(rows, per_col, rng):
    """+-1 on per_col rows of every column, all rows used about equally."""
    W = np.zeros((rows, H))
    order = np.concatenate([rng.permutation(rows) for _ in range(-(-per_col * H // rows))])
    for j in range(H):
        W[order[j * per_col:(j + 1) * per_col], j] = rng.choice([-1.0, 1.0], per_col)
    return W


def _signs(count, share, rng):
    """k in {-1, 0, 1}, never 0 next to the ends of 16, 64 and 2048 nodes."""
    j = np.arange(count)
    k = rng.choice([-1.0, 1.0], count) * (rng.random(count) < share)
    edge = (j % 2048 < 2) | (j % 2048 > 2045) | (j >= count - 3) | (j % 1024 == 511)
    return np.where(edge & (k == 0), rng.choice([-1.0, 1.0], count), k)


def instance(m, n, layers, seed):
    rng = np.random.default_rng(seed)
    A = _graph(m, n, 3 if layers == 1 else 1, rng)
    ints = lambda lo, hi, k: rng.integers(lo, hi + 1, k).astype(np.float64)  # noqa: E731
    vlo = np.where(rng.random(n) < 0.3, -np.inf, ints(-1, 0, n))
    vhi = np.where(rng.random(n) < 0.3, np.inf, ints(1, 2, n))
    clo = np.where(rng.random(m) < 0.3, -np.inf, ints(-1, 1, m))
    chi = np.where(rng.random(m) < 0.3, np.inf, np.where(np.isfinite(clo), clo, 0) + ints(0, 2, m))
    lp = lpgen.LP(m, n, A.indptr.astype(np.int32), A.indices.astype(np.int32), A.data,
                  ints(-1, 1, n), clo, chi, vlo, vhi, name=f"exact{m}x{n}")
    per = 8 if layers == 1 else 2
    w = [np.where(rng.random(H) < 0.1, 2 * ints(129, 255, H) - 1, ints(1, 2, H)) * rng.choice([-1, 1], H)
         for _ in range(2)]
    p = gnn_ref.pack(dict(
        W_cin=_weights(F, 3, rng), W_rin=_weights(F, 3, rng),
        W_c=[_weights(2 * H, per, rng) for _ in range(layers)],
        W_r=[_weights(2 * H, per, rng) for _ in range(layers)], w_x=w[0], w_y=w[1]))
    ref = dict(c=ints(-1, 1, n), b=ints(-1, 1, m), x=ints(-2, 2, n), y=ints(-2, 2, m))
    X = gnn_ref.features(lp.c, clo, chi, vlo, vhi, ref["c"], ref["b"], ref["x"], ref["y"],
                         np.ones(m), np.ones(n))
    px, py, _ = gnn_ref.forward(p, layers, A, *X, ref["x"], ref["y"])
    share = min(1.0, 600.0 / max(m, n))
    tx, ty = px - n * _signs(n, share, rng), py - m * _signs(m, share, rng)
    return dict(lp=lp, A=A, p=p, ref=ref, X=X, px=px, py=py, tx=tx, ty=ty, layers=layers)


def check_exact(I):
    """Raises if a number of the instance's forward or backward pass is not
    held exactly (see the head of this file)."""
    A, layers, At, absA = I["A"], I["layers"], I["A"].T.tocsr(), abs(I["A"])
    W = gnn_ref.unpack(I["p"], layers)
    px, py, c = gnn_ref.forward(I["p"], layers, A, *I["X"], I["ref"]["x"], I["ref"]["y"])
    lim = lambda v, what: _lim(np.abs(v).max(initial=0.0), 2.0 ** 24, what)  # noqa: E731
    for name in ("Hc0", "Hr0"):
        assert (bf16(c[name]) == c[name]).all(), name
    for name in ("INc", "INr", "Hc", "Hr"):
        for v in c[name]:
            assert (bf16(v) == v).all() and (v == np.rint(v)).all(), name
    for k in ("W_cin", "W_rin"):
        assert (bf16(W[k]) == W[k]).all()
    for v, h, w in ((px, c["Hc"][-1], W["w_x"]), (py, c["Hr"][-1], W["w_y"])):
        lim(np.abs(h) @ np.abs(w) + 2, "prediction")
    lim(I["tx"], "target"), lim(I["ty"], "target")
    dx, dy = 2 * (px - I["tx"]) / px.size, 2 * (py - I["ty"]) / py.size
    assert (dx == np.rint(dx)).all() and (dy == np.rint(dy)).all()
    lim(np.abs(c["Hc"][-1]).T @ np.abs(dx), "head"), lim(np.abs(c["Hr"][-1]).T @ np.abs(dy), "head")
    dHc, dHr = np.outer(dx, W["w_x"]), np.outer(dy, W["w_y"])
    low = 0

    def pair(dZ):
        nonlocal low
        hi = bf16(dZ)
        lo = dZ - hi
        assert (bf16(lo) == lo).all(), "gradient pair"
        low += int((lo != 0).sum())
        return np.abs(hi) + np.abs(lo)

    def back(dH, Hl, IN, Wl):
        dZ = dH * (Hl > 0)
        a = pair(dZ)
        lim(np.abs(IN).T @ a, "weight gradient")
        lim(a @ np.abs(Wl).T, "data gradient")
        return dZ @ Wl.T

    for l in range(layers - 1, -1, -1):
        gc = back(dHc, c["Hc"][l], c["INc"][l], W["W_c"][l])
        lim(absA @ np.abs(gc[:, H:]) + np.abs(dHr), "row products")
        dHr = dHr + A @ gc[:, H:]
        gr = back(dHr, c["Hr"][l], c["INr"][l], W["W_r"][l])
        lim(absA.T @ np.abs(gr[:, H:]) + np.abs(gc[:, :H]), "column products")
        dHc, dHr = gc[:, :H] + At @ gr[:, H:], gr[:, :H]
    lim(np.abs(I["X"][0]).T @ pair(dHc * (c["Hc0"] > 0)), "embedding")
    lim(np.abs(I["X"][1]).T @ pair(dHr * (c["Hr0"] > 0)), "embedding")
    assert low > 0, "no gradient needs its low half"


def _lim(v, bound, what):
    assert v < bound, (what, float(v))


# m, n, layers, seed (a seed whose instance passes check_exact): one node, the
# edges of 16 nodes per wave, 64 per step and 2048 per chunk of the weight
# gradients, one to seven chunks, the node counts around which the layer update
# takes its other form, and more nodes than one round of its workgroups holds
CASES = [(1, 1, 1, 1), (1, 1, 2, 1), (5, 16, 1, 1), (17, 33, 2, 1), (64, 63, 1, 1), (65, 2047, 2, 2),
         (2049, 2048, 1, 1), (4096, 640, 1, 2), (4097, 700, 2, 2), (6145, 2050, 1, 1),
         (12287, 12289, 1, 1), (12288, 12288, 2, 2), (33000, 40001, 1, 1), (40000, 32790, 2, 1)]
