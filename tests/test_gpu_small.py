"""The 2D Poisson grids that one workgroup per right-hand side runs alone (sides
up to 128 above a coarsest side of at most 64): one preconditioned step against a
NumPy V-cycle, and whole solves against the sine-transform oracle, at the edges of
the strips (sides at and beside 32, 64 and 128, odd coarsest sides, one unknown)."""
import ctypes

import numpy as np
import pytest

from oracle import operators
from tests.gpu_util import from_dev, require_gpu, to_dev

pytestmark = pytest.mark.gpu

GRIDS = [(2, 2), (6, 2), (30, 2), (32, 3), (34, 2), (62, 2), (64, 2), (64, 4), (66, 2), (100, 3),
         (126, 2), (128, 2), (128, 5), (128, 8)]


def _nb_sum(x):
    s = np.zeros_like(x)
    s[:, 1:] += x[:, :-1]
    s[:, :-1] += x[:, 1:]
    s[:, :, 1:] += x[:, :, :-1]
    s[:, :, :-1] += x[:, :, 1:]
    return s


def _vcycle(b, d, c, levels, pre, post, omega, cycles=1, top=False, x=None):
    """x + V(b - A x) on grids b [m, N, N]; exact coarsest solve."""
    N = b.shape[1]
    if levels == 1:
        B = b.reshape(len(b), -1).T
        return operators.poisson2d_solve_dst(N, B, d, c).T.reshape(b.shape)
    red = (np.add.outer(np.arange(N), np.arange(N)) % 2 == 0)[None]
    x = np.zeros_like(b) if x is None else x
    for _ in range(pre):
        for m in (red, ~red):
            x = np.where(m, (b + c * _nb_sum(x)) / d, x)
    r = b - (d * x - c * _nb_sum(x))
    rc = 0.5 * r.reshape(len(b), N // 2, 2, N // 2, 2).sum(axis=(2, 4))
    e = None
    for _ in range(cycles if top and levels > 2 else 1):
        e = _vcycle(rc, d - 2 * c, c / 2, levels - 1, pre, post, omega, x=e)
    x = x + 0.5 * omega * np.repeat(np.repeat(e, 2, axis=1), 2, axis=2)
    for _ in range(post):
        for m in (~red, red):
            x = np.where(m, (b + c * _nb_sum(x)) / d, x)
    return x


def _est(N, L, **kw):
    require_gpu()
    import paper_2108_11281_amd as m
    kw.setdefault("nb", 8)
    kw.setdefault("solve_tol", 1e-12)
    return m.TraceEstimator("poisson2d", N, L, **kw)


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("N,L", GRIDS)
def test_one_step_is_the_vcycle(N, L, precision):
    # one CG iteration returns alpha M b with alpha = b^T M b / (M b)^T A (M b)
    rng = np.random.default_rng(N + L)
    b = rng.standard_normal((3, N, N))
    sweeps = [(1, 1, 1), (2, 2, 2)] + ([(0, 1, 1), (2, 0, 1), (3, 2, 2)] if N in (34, 100) else [])
    for pre, post, cyc in sweeps:
        est = _est(N, L, precision=precision, nu_pre=pre, nu_post=post, top_cycles=cyc, omega=1.8,
                   max_iter=1, max_refine=1)
        z = _vcycle(b, 4.0, 1.0, L, pre, post, 1.8, cyc, True)
        Az = 4.0 * z - _nb_sum(z)
        ref = (b * z).sum(axis=(1, 2)) / (z * Az).sum(axis=(1, 2))
        ref = ref[:, None, None] * z
        B = to_dev(b.reshape(3, -1))
        Y = est._vec(1, 3)
        rc = est._lib.mlmc_solve(est._ctx, 1, 3, ctypes.c_void_p(B.data_ptr()),
                                 ctypes.c_void_p(Y.data_ptr()), None)
        assert rc in (0, -4)
        # FP64: 1e-12 relative; FP32: 1e-4, the rounding of some hundred operations
        # per unknown times the V-cycle's conditioning
        tol = 1e-12 if precision == "fp64" else 1e-4
        got = from_dev(Y).reshape(b.shape)
        assert np.max(np.abs(got - ref)) <= tol * np.max(np.abs(ref)), (pre, post, cyc)
        est.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("N,L", GRIDS)
def test_solves_match_the_sine_transform(N, L, precision):
    est = _est(N, L, precision=precision, diag=4.1, off=1.0)
    rng = np.random.default_rng(7)
    d, c = 4.1, 1.0
    for l in range(1, L + 1):
        S = N >> (l - 1)
        b = rng.standard_normal((5, S * S))
        b[2] *= 1e-6      # columns of different scale converge on their own
        b[4] = 0.0
        Y, rel = est.solve(l, to_dev(b))
        assert np.all(rel <= 1e-12)
        ref = operators.poisson2d_solve_dst(S, b.T, d, c).T
        lam = d - 4.0 * c * np.cos(np.pi / (S + 1))
        # |y - A^-1 b| = |A^-1 r| <= |r| / lambda_min, and the rounding of the oracle
        err = np.linalg.norm(from_dev(Y) - ref, axis=1)
        bn = np.linalg.norm(b, axis=1)
        assert np.all(err <= (1e-12 + 1e-14) * bn / lam + 1e-13 * np.linalg.norm(ref, axis=1)), l
        d, c = d - 2 * c, c / 2
    est.close()
