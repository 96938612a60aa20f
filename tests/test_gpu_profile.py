"""psara_profile_passes times the launch that the iterations run in place of P6 and P7: the fused pass
with the coarse levels (paired), the fused pass alone (initialisation), or none (a large image); the
state advances by 2 * iters iterations with the bits of a solve."""
import numpy as np
import pytest

from paper_1801_02417_amd import workloads as wk
from tests.gpu_common import P, say, solver_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec,shapes,one", [(64, "fp32", None, True), (64, "fp64", None, True),
                                               (128, "fp32", {"fft_cells": 1024}, False),
                                               (512, "fp32", None, False), (256, "fp64", None, False)])
def test_the_launch_of_p6_and_p7(n, prec, shapes, one):
    M, rng = 6001, np.random.default_rng(n)
    uv = wk.gaussian_uv(rng, M)
    Y = rng.standard_normal((M, 4)) + 1j * rng.standard_normal((M, 4))

    def make():
        s = solver_for(uv, n, 8, prec, levels=3, gamma=1e-3)
        s.set_data(Y, 0.3 * float(np.linalg.norm(Y)))
        s.opnorm(30, 1e-2)
        s.set_steps(*P.psara_step_sizes(0, 1.3 * s.phi_norm_sq))
        s.set_tuning(shapes)
        return s

    s, ref = make(), make()
    try:
        ms = s.profile_passes(P.PSARA_CONSTRAINED, 4)
        say(f"[profile] n={n} {prec} {shapes}: P6 {ms[5]:.4f} P7 {ms[6]:.4f} one launch {ms[10]:.4f} ms")
        assert (ms[10] > 0) == one
        assert min(ms[i] for i in (0, 1, 4, 5, 6, 7, 8, 9)) > 0
        ref.solve(P.PSARA_CONSTRAINED, 8, report=False)
        a, b = s.state(), ref.state()
        for k in a:
            assert np.array_equal(a[k], b[k]), k
        assert s.profile_passes(P.PSARA_NNLS_INIT, 2)[10] > 0
    finally:
        s.close()
        ref.close()


def test_paired_launch_holds_the_coarse_levels():
    """At 256^2 with few rows the coarse levels are the longer part of the paired launch: its time is
    theirs, several times that of the fused pass alone."""
    n, M, rng = 256, 2001, np.random.default_rng(3)
    s = solver_for(wk.gaussian_uv(rng, M), n, 8, "fp32", levels=4, gamma=1e-3)
    try:
        s.set_data(np.ones((M, 4), complex), 1.0)
        s.opnorm(30, 1e-2)
        s.set_steps(*P.psara_step_sizes(0, 1.3 * s.phi_norm_sq))
        s.profile_passes(P.PSARA_CONSTRAINED, 4)
        paired, alone = (s.profile_passes(m, 16)[10] for m in (P.PSARA_CONSTRAINED, P.PSARA_NNLS_INIT))
        say(f"[profile] paired {paired * 1e3:.1f} us, fused alone {alone * 1e3:.1f} us")
        assert paired > 1.5 * alone
    finally:
        s.close()
