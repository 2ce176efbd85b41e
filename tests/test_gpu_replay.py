"""Graph replay of the runs between checks for short check periods (runs of 0,
1, 2, ... iterations, in front of them one eager iteration or a fresh epoch's
check), bitwise against eager launches, with the program's own work on the
stream between the calls, and the control block's scalars after every call."""
import numpy as np
import pytest

import lpgen
from tests.test_gpu_parity import D  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("period", [1, 2, 3, 4, 7, 64])
@pytest.mark.parametrize("precision", [0, 1])
def test_replay_matches_eager_for_short_periods(D, period, precision):  # noqa: F811
    import torch
    lp = lpgen.config0()
    states = []
    for graphs in (0, 1):
        G = D.Problem(lp, eps=0.0, check_period=period, use_graphs=graphs, precision=precision,
                      stream=torch.cuda.current_stream())
        G.init()
        out = []
        for n in (5 * period, 3, 2 * period + 1, 6 * period):
            G.iterate(n)
            torch.ones(1000, device="cuda").sum().item()      # work between the replays
            k = G.kkt()                                       # leaves the solver's state alone
            s = G.state()
            out.append({q: s[q].copy() for q in ("x", "y", "xa", "ya", "xh", "yh")} | {
                "scalars": np.array([float(v) for v in s["scalars"].values()]), "kkt": k})
        states.append(out)
    for a, b in zip(*states):
        for q in a:
            assert np.array_equal(a[q], b[q]), (period, q)
