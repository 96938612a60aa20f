"""psara_opnorm: the quotients of the power iteration at step counts around a round of queued steps
grow towards the largest eigenvalue of Re phi^dagger phi (from the oracle, in 64 bits) and never
beyond it; a loose test stops at the step at which it first holds; for every tap count, with fewer
and more rows than a round needs, FP32 and FP64 contexts (the iteration itself is always FP64)."""
import time

import numpy as np
import pytest

from oracle import problem
from paper_1801_02417_amd import workloads as wk
from tests.gpu_common import P, say, solver_for

pytestmark = pytest.mark.gpu


def _largest(mop, n):
    """The largest eigenvalue of the symmetric 4n^2 x 4n^2 matrix of Re phi^dagger phi."""
    N = n * n
    A = np.zeros((4 * N, 4 * N))
    for j in range(4 * N):
        x = np.zeros((N, 4))
        x.flat[j] = 1.0
        A[:, j] = np.real(mop.phi_adj(mop.phi(x))).ravel()
    return float(np.linalg.eigvalsh(0.5 * (A + A.T))[-1])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("taps,M", [(4, 40), (6, 200), (8, 1), (8, 700)])
def test_quotients_grow_to_the_norm(taps, M, prec):
    n = 8
    wl = wk.tiny(n=n, M=M, taps=taps, levels=1, seed=M)
    b = problem.build(wl, norm_rtol=1e-3, norm_max_iter=4)
    top = _largest(b.mop, n)
    s = solver_for(wl, n, taps, prec, levels=1, gamma=b.gamma)
    try:
        q = [s.opnorm(k, 0.0) for k in (1, 2, 7, 8, 9, 15, 16, 17, 400)]
        say(f"[opnorm] taps={taps} M={M} {prec}: {q[0]:.6g} .. {q[-1]:.6g}, exact {top:.6g}")
        # FP64 rounding of the quotients: sums of a few hundred products, well inside 1e-12
        assert all(y >= x * (1 - 1e-12) for x, y in zip(q, q[1:])), q
        assert q[-1] <= top * (1 + 1e-10) and q[-1] >= top * (1 - 2e-2), (q[-1], top)
        steps = [s.opnorm(k, 0.0) for k in range(1, 12)]
        first = next(k for k in range(1, 11) if abs(steps[k] - steps[k - 1]) <= 0.05 * steps[k])
        assert s.opnorm(500, 0.05) == steps[first]
    finally:
        s.close()


def _best(f, n=7):
    best = 1e9
    for _ in range(n):
        t = time.perf_counter()
        f()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("stop", [2, 3, 5, 9])
def test_a_loose_test_costs_the_steps_it_takes(stop):
    """The steps queued beyond the one that meets the test must not run: the call takes the time of as
    many steps with the test off (some 0.3 ms each here), and half as much again at most."""
    wl = wk.ring256()
    s = P.Solver(wl.n, wl.uv, taps=wl.taps, precision=P.PSARA_FP64)
    try:
        q = [s.opnorm(k, 0.0) for k in range(1, stop + 1)]
        rtol = 1.0 if stop == 2 else abs(q[-1] / q[-2] - 1.0) * q[-2] / q[-1] * (1.0 + 1e-9)
        assert s.opnorm(500, rtol) == q[-1]
        fixed, loose = _best(lambda: s.opnorm(stop, 0.0)), _best(lambda: s.opnorm(500, rtol))
        say(f"[opnorm] stop at step {stop}: {loose * 1e3:.2f} ms, {stop} steps {fixed * 1e3:.2f} ms")
        assert loose <= 1.5 * fixed
        s.set_prior(4, 1e-3)
        s.set_data(np.ones((wl.M, 4), complex), 1.0)
        s.opnorm(500, rtol)
        s.set_steps()
        s.solve(P.PSARA_NNLS_INIT, 3, report=False)
        assert np.any(s.image())                          # nothing is left halted
    finally:
        s.close()
