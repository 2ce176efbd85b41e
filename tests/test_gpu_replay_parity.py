"""Graph replays held to the oracle and to eager launches where a replay is
known to happen: a handle replays from its third complete run between two
checks on, so every case here has more runs than that, before and after a
change of what the graph holds (diag(Q), the check period, gamma), and at the
full sizes of the benchmark workloads (sliced formats, non-temporal streams).

Bars: replays launch the kernels of the eager runs on the same data, so they
are equal bit for bit; against the oracle the parity tests' 1e-10."""
import dataclasses
import functools

import numpy as np
import pytest

import lpgen
from tests.test_gpu_parity import D, O, compare_iterates, compare_logs, gpu_params, rel  # noqa: F401

pytestmark = pytest.mark.gpu
PERIOD = 8


def start(D, O, lp):  # noqa: F811
    """Oracle and library at the same start, with PERIOD between the checks."""
    P0 = O.Problem(lp)
    kw = dict(eta=P0.eta, omega0=P0.omega0, eps=0.0, check_period=PERIOD)
    P = O.Problem(lp, O.Params(**kw))
    st = P.init_state()
    G = D.Problem(lp, gpu_params(D, **kw))
    G.init()
    return P, st, G, kw


def both(P, st, G, n, params=None):
    P.run(st, n, params)
    G.iterate(n)
    assert compare_logs(G.log(), st["log"]) is None
    compare_iterates(G.state(), st, 1e-10)


def test_diag_set_and_cleared_between_replays(D, O):  # noqa: F811
    """The primal step's kernel is a node of the graph: after diag(Q) is set,
    and after it is taken back, the replays run the other step."""
    qp = lpgen.constructed_qp(1000, 2000, 500, 4, seed=29)
    lp = dataclasses.replace(qp, q=None)
    P, st, G, _ = start(D, O, lp)
    plain = P.init_state()
    both(P, st, G, 10 * PERIOD + 3)
    O.lib().ora_set_qdiag(P._h, qp.q.ctypes.data)
    G.set_objective_diag(qp.q)
    both(P, st, G, 8 * PERIOD)
    # replays of the earlier step would end elsewhere
    O.lib().ora_set_qdiag(P._h, None)
    P.run(plain, 18 * PERIOD + 3)
    assert rel(plain["x"], st["x"]) > 1e-3
    G.set_objective_diag(None)
    both(P, st, G, 8 * PERIOD)


@pytest.mark.parametrize("change", [dict(check_period=12), dict(check_period=5),
                                    dict(check_period=1), dict(gamma=0.7)])
def test_set_params_between_replays(D, O, change):  # noqa: F811
    """The number of iterations of a run and gamma are in the graph."""
    lp = lpgen.constructed_lp(1500, 3000, 750, 4, seed=31)
    P, st, G, kw = start(D, O, lp)
    both(P, st, G, 10 * PERIOD + 3)
    old = {k: (v.copy() if isinstance(v, np.ndarray) else v) for k, v in st.items() if k != "state"}
    old["state"] = type(st["state"]).from_buffer_copy(st["state"])
    old["log"] = list(st["log"])
    G.set_params(**change)
    both(P, st, G, 90, O.Params(**{**kw, **change}))
    P.run(old, 90)
    assert rel(old["x"], st["x"]) > 1e-8            # the change shows


@functools.lru_cache(maxsize=1)
def instance(name):
    return {"c1": lpgen.config1, "staircase": lpgen.config1_staircase,
            "lasso": lambda: lpgen.lasso_qp(1_000_000, 500_000, 20, seed=7)}[name]()


@pytest.mark.slow
@pytest.mark.parametrize("name,fp32", [("c1", False), ("c1", True), ("staircase", False), ("lasso", False)])
def test_fullsize_replays_match_eager(D, name, fp32):  # noqa: F811
    """261 iterations at the default period of 64: the runs from t = 129 and
    t = 193 are replayed."""
    lp = instance(name)
    out = []
    for graphs in (0, 1):
        G = D.Problem(lp, gpu_params(D, eta=0.9, omega0=1.0, eps=0.0, use_graphs=graphs,
                                     precision=D.FP32_MIXED if fp32 else D.FP64,
                                     fp32_switch_tol=0.0, fp32_stall_checks=10**6, fp32_diverge=0.0))
        G.init()
        G.iterate(261)
        out.append((G.state(), G.log()))
        G.close()
    (a, la), (b, lb) = out
    assert len(la) == len(lb) >= 5 and la == lb
    for k in ("x", "y", "xa", "ya", "xh", "yh"):
        assert np.isfinite(a[k]).all() and np.array_equal(a[k], b[k]), k
    assert a["scalars"] == b["scalars"]
