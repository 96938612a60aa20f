"""P6 and P7 as two passes and as one fused pass give the same bits, so that a launch may take either:
the paired launches of a solve with the default shapes (fused) against the launches on two streams
that more FFT cells per workgroup ask for (two passes, or fused where the chunks are full; at 256^2 in
FP32 the coarse levels begin one level later there), and members of a batch too large for the paired launches against their runs alone.  Chunks of every kind
(of one row, up to and beyond the sizes that one wave grids and that eight lanes to a row de-grid, of
runs), every tap count, known Mueller matrices, both precisions."""
import numpy as np
import pytest

from paper_1801_02417_amd import workloads as wk
from tests.gpu_common import P, say, solver_for

pytestmark = pytest.mark.gpu


def _member(n, uv, taps, levels, prec, seed, mueller):
    rng = np.random.default_rng(seed)
    M = len(uv)
    s = solver_for(uv, n, taps, prec, levels=levels, gamma=1e-3)
    if mueller:
        P.psara_set_mueller(s.ctx, wk.station_mueller(np.random.default_rng(5), M))
    Y = rng.standard_normal((M, 4)) + 1j * rng.standard_normal((M, 4))
    s.set_data(Y, 0.3 * float(np.linalg.norm(Y)))
    s.opnorm(30, 1e-2)
    s.set_steps(*P.psara_step_sizes(0, 1.3 * s.phi_norm_sq))
    return s


def _uv(n, rng, sizes):
    """Window starts that fill gridding tiles with the given row counts, every third tile with rows of
    one window start (runs), in tiles spread over the grid."""
    K, side = 2 * n, max(1, 2 * n // 16)
    uv = []
    for i, rows in enumerate(sizes):
        t = (i * 7) % (side * side)
        a, b = divmod(t, side)
        if i % 3 == 2:
            at = np.array([[16 * a + 5.25, 16 * b + 9.5]]) + rng.uniform(0.0, 0.2, size=(rows, 2))
        else:
            at = rng.uniform(0.0, 16.0, size=(rows, 2)) + np.array([16.0 * a, 16.0 * b])
        uv.append((at / K * 2 * np.pi + np.pi) % (2 * np.pi) - np.pi)
    return np.clip(np.concatenate(uv), -np.pi, np.pi - 1e-9)


SIZES = [1, 7, 8, 9, 16, 17, 31, 63, 64, 65, 100, 130, 200, 300]


def _run(s, mode):
    s.solve(P.PSARA_NNLS_INIT, 3, report=False)
    s.solve(mode, 9, report=False)
    return s.state()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,taps,levels,sizes,mueller,mode", [
    (64, 8, 3, SIZES, False, "CONSTRAINED"),
    (64, 6, 4, SIZES, True, "UNCONSTRAINED"),
    (128, 4, 2, SIZES + [700], False, "CONSTRAINED"),
    (16, 8, 1, [900, 1100, 1024, 500], False, "CONSTRAINED"),      # full chunks
    (32, 8, 2, [40] * 16, True, "CONSTRAINED"),
    (256, 8, 4, SIZES, False, "CONSTRAINED"),                      # another first coarse level, too
    (256, 8, 3, [1000] * 40, False, "CONSTRAINED"),
])
def test_routes_give_the_same_bits(n, taps, levels, sizes, mueller, mode, prec):
    uv = _uv(n, np.random.default_rng(n + taps), sizes)
    s = _member(n, uv, taps, levels, prec, 0, mueller)
    try:
        out = {}
        for cells in (0, 1024, 2048):
            s.set_tuning({"fft_cells": cells})
            s.reset()
            out[cells] = _run(s, getattr(P, "PSARA_" + mode))
    finally:
        s.close()
    assert float(np.abs(out[0]["B"]).max()) > 0.0
    for cells in (1024, 2048):
        for k in out[0]:
            assert np.array_equal(out[0][k], out[cells][k]), (n, taps, prec, cells, k)
    say(f"[routes] n={n} taps={taps} {prec}: bitwise equal")


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_large_batch_equals_alone(prec):
    """30 members of some 72 chunks each."""
    n, taps, levels, count = 64, 8, 3, 30
    uv = _uv(n, np.random.default_rng(4), SIZES * 4)
    members = [_member(n, uv, taps, levels, prec, i % 2, False) for i in range(count)]
    try:
        P.batch_solve(members, P.PSARA_NNLS_INIT, 3, report=False)
        P.batch_solve(members, P.PSARA_CONSTRAINED, 9, report=False)
        batched = [s.state() for s in members]
    finally:
        for s in members:
            s.close()
    for i in range(2):
        s = _member(n, uv, taps, levels, prec, i, False)
        try:
            alone = _run(s, P.PSARA_CONSTRAINED)
        finally:
            s.close()
        for j in range(i, count, 2):
            for k in alone:
                assert np.array_equal(alone[k], batched[j][k]), (prec, j, k)
