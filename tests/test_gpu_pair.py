"""Iterations whose prior branch runs inside the data branch's launches: at most one analysis level
before the coarse ones (sides up to 256 in FP32, 128 in FP64), for every tap count; against the
oracle from a random state, to the bars of the iteration tests.  Batches of such sides, alone and
mixed with a larger one, equal their members run alone, bitwise."""
import numpy as np
import pytest

from oracle import problem
from paper_1801_02417_amd import workloads as wk
from tests.gpu_common import P, say, solver_for
from tests.test_gpu_iteration import _compare, _oracle_steps, _random_state

pytestmark = pytest.mark.gpu


def _problem(n, M, taps, levels):
    wl = wk.tiny(n=n, M=M, taps=taps, levels=levels, seed=n + M)
    b = problem.build(wl, norm_rtol=1e-3, norm_max_iter=8)
    b.pb.tau *= 0.5                      # a rough operator norm, so steps well inside their bound
    return wl, b


def _solver(wl, b, prec, W=None):
    s = solver_for(wl, wl.n, wl.taps, prec, levels=wl.levels, gamma=b.gamma, weights=W)
    s.set_data(b.pb.Y, b.pb.eps)
    s.opnorm(20, 1e-6)
    s.set_steps(b.pb.tau, b.pb.rho1, b.pb.rho2, b.pb.rho3)
    return s


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("fp32", 2e-6)])
@pytest.mark.parametrize("n,M,taps,levels", [(8, 7, 4, 1), (16, 37, 6, 2), (32, 601, 8, 3), (64, 1511, 4, 1),
                                             (64, 6000, 8, 4), (128, 3001, 6, 2), (256, 2001, 8, 3)])
def test_paired_iterations(n, M, taps, levels, prec, tol):
    wl, b = _problem(n, M, taps, levels)
    W = np.random.default_rng(n).uniform(0.2, 1.0, size=(b.sara.J, 4))
    s = _solver(wl, b, prec, W)
    try:
        gW = b.gamma * W
        st = _random_state(np.random.default_rng(3), n * n, b.sara.J, M, gW)
        s.set_state(st.S, st.Z, st.A, st.B, st.C, st.D)
        ref, scale = st.copy(), {}
        for k in (1, 3):
            s.solve(P.PSARA_CONSTRAINED, k, report=False)
            ref = _oracle_steps(ref, b.pb, gW, "polsara", k, scale)
            w = _compare(s.state(), ref, tol, f"n={n} taps={taps} {prec} +{k}", scale if prec == "fp32" else None)
            say(f"[pair] n={n} M={M} taps={taps} levels={levels} {prec} +{k}: worst rel err {w:.2e}")
    finally:
        s.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("largest", [(64, 1511, 4), (256, 2001, 4), (512, 2001, 4)])
def test_paired_batch_equals_alone(largest, prec):
    probs = [_problem(n, M, 8, lv) for n, M, lv in [(16, 37, 2), largest, (32, 601, 3)]]
    members = [_solver(wl, b, prec) for wl, b in probs]
    try:
        P.batch_reweighted_solve(members, P.PSARA_CONSTRAINED, [9, 7])
        batched = [s.image() for s in members]
    finally:
        for s in members:
            s.close()
    for (wl, b), img in zip(probs, batched):
        s = _solver(wl, b, prec)
        s.reweighted_solve(P.PSARA_CONSTRAINED, [9, 7])
        assert np.array_equal(s.image(), img), (wl.n, largest, prec)
        s.close()
