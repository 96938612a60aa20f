"""The default gridding chunk size: row counts on both sides of the rule's lines (one tile of up to 4
and of more than 4 smallest chunks; problems with few and many tiles), two iterations from a random
state against the oracle, to the bars of the iteration tests, at the default and at an explicit
size."""
import numpy as np
import pytest

from tests.gpu_common import P, say
from tests.test_gpu_iteration import _compare, _oracle_steps, _random_state
from tests.test_gpu_pair import _problem, _solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 2e-6)])
@pytest.mark.parametrize("n,M", [(8, 64), (8, 65), (8, 256), (8, 257), (8, 1025), (8, 4097), (64, 900), (256, 2500)])
def test_iterations_at_chunk_edges(n, M, prec, tol):
    wl, b = _problem(n, M, 8, 1 if n == 8 else 4)
    W = np.random.default_rng(n).uniform(0.2, 1.0, size=(b.sara.J, 4))
    gW = b.gamma * W
    st = _random_state(np.random.default_rng(3), n * n, b.sara.J, M, gW)
    scale = {}
    ref = _oracle_steps(st.copy(), b.pb, gW, "polsara", 2, scale)
    for tuning in (None, {"grid_chunk": 256}):
        s = _solver(wl, b, prec, W)
        try:
            if tuning:
                s.set_tuning(tuning)
            s.set_state(st.S, st.Z, st.A, st.B, st.C, st.D)
            s.solve(P.PSARA_CONSTRAINED, 2, report=False)
            w = _compare(s.state(), ref, tol, f"n={n} M={M} {prec} {tuning}", scale if prec == "fp32" else None)
            say(f"[chunks] n={n} M={M} {prec} {tuning}: worst rel err {w:.2e}")
        finally:
            s.close()
