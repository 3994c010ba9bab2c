"""2D Poisson solves by lockstep launches (top sides above 128, or a coarsest side above
64): solutions of a batch against the sine-transform oracle on ragged sides, for right-hand
sides that are FP32 numbers and that are not, with a zero column and columns of different
smoothness and scale, which converge after different numbers of refinements (the FP64
iterate alternates between two planes, so their results lie in different ones)."""
import numpy as np
import pytest

from oracle import operators
from tests.gpu_util import from_dev, require_gpu, to_dev

pytestmark = pytest.mark.gpu

# 130 over 65, 200 over 100 and 50, 264 over 132, 66 and 33
GRIDS = [(130, 2), (200, 3), (264, 4)]
TOL = 1e-12


def _columns(N, count, fp32):
    rng = np.random.default_rng(N + count)
    if fp32:  # probes
        b = rng.choice([-1.0, 1.0], (count, N * N))
        if count > 4:
            b[4] *= 2.0 ** -20
        return b
    b = rng.standard_normal((count, N * N))
    if count > 1:
        b[1] = 0.0
    if count > 2:  # the smoothest mode
        s = np.sin(np.pi * np.arange(1, N + 1) / (N + 1))
        b[2] = np.outer(s, s).ravel()
    if count > 3:  # a single cell
        b[3] = 0.0
        b[3, N * (N // 2) + N // 3] = 1.0 / 3.0
    if count > 4:
        b[4] *= 1e-6
    return b


def _check(est, N, b):
    Y, rel = est.solve(1, to_dev(b))
    assert np.all(rel <= TOL)
    ref = operators.poisson2d_solve_dst(N, b.T, 4.1, 1.0).T
    lam = 4.1 - 4.0 * np.cos(np.pi / (N + 1))
    err = np.linalg.norm(from_dev(Y) - ref, axis=1)
    bn = np.linalg.norm(b, axis=1)
    # |y - A^-1 b| <= |r| / lambda_min, and the rounding of the oracle
    assert np.all(err <= (TOL + 1e-14) * bn / lam + 1e-13 * np.linalg.norm(ref, axis=1)), err


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("N,L", GRIDS)
def test_solutions_match_the_sine_transform(N, L, precision):
    require_gpu()
    import paper_2108_11281_amd as m
    for sweeps in (1, 2):
        est = m.TraceEstimator("poisson2d", N, L, diag=4.1, off=1.0, precision=precision, nb=9,
                               solve_tol=TOL, nu_pre=sweeps, nu_post=sweeps)
        for count in (1, 5, 9):
            for fp32 in (False, True):
                _check(est, N, _columns(N, count, fp32))
        est.close()


@pytest.mark.parametrize("N,L", GRIDS)
def test_columns_that_stop_at_different_refinements(N, L):
    require_gpu()
    import paper_2108_11281_amd as m
    b = _columns(N, 9, False)
    mixed = []
    for inner_tol in (1e-1, 1e-2, 1e-3, 1e-4):
        est = m.TraceEstimator("poisson2d", N, L, diag=4.1, off=1.0, precision="fp32_ir64", nb=9,
                               solve_tol=TOL, nu_pre=1, nu_post=1, inner_tol=inner_tol)
        refinements = []
        for k in range(len(b)):
            est.solve(1, to_dev(b[k:k + 1]))
            refinements.append(est.counters()[1])
        # the last refinement of some columns is an odd one, of others an even one
        mixed.append({r % 2 for r in refinements} == {0, 1})
        _check(est, N, b)
        est.close()
    assert any(mixed)
