"""The FFT passes at every line length (sides 8 to 1024, so grid lines of 16 to 2048 cells, with one or
several lines to a workgroup and a last workgroup that is not full) and every cell count per
workgroup that the side allows: phi and phi^dagger against the FP64 oracle, to the bars of the
operator tests."""
import numpy as np
import pytest

from oracle.nufft import NUFFT, MeasurementOp
from tests.gpu_common import P, random_uv, rel_err, say, solver_for
from tests.test_gpu_operators import TOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8, 16, 32, 64, 128, 256, 512, 1024])
def test_operators_at_every_line_length(n):
    rng = np.random.default_rng(n)
    uv = random_uv(rng, 61)
    mop = MeasurementOp(NUFFT(uv, n, 2, 6))
    S = rng.standard_normal((n * n, 4))
    B = rng.standard_normal((61, 4)) + 1j * rng.standard_normal((61, 4))
    y, x = mop.phi(S), np.real(mop.phi_adj(B))
    for prec in ("fp64", "fp32"):
        s = solver_for(uv, n, 6, prec)
        try:
            for cells in (0, 512, 1024, 2048):
                if 0 < cells < 2 * n:
                    continue
                s.set_tuning({"fft_cells": cells})
                e1, e2 = rel_err(s.phi(S), y), rel_err(s.phi_adjoint(B), x)
                say(f"[fft] n={n} {prec} cells={cells}: phi {e1:.2e} adjoint {e2:.2e}")
                assert e1 <= TOL[prec] and e2 <= TOL[prec]
        finally:
            s.close()
