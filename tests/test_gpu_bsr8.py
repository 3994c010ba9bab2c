"""Levels with eight complex unknowns per site (matrix-core block kernels): operator,
sweeps, restriction and reported residuals at the edges of the column groups, on
hierarchies whose restrictions take the matrix cores or (rows of four fine unknowns) not, against sparse matrices formed from the exported prolongations."""
import ctypes

import numpy as np
import pytest
import scipy.sparse as sp

from oracle import hierarchy, operators
from tests.gpu_util import from_dev, require_gpu, to_dev
from workloads import gauge_field

pytestmark = pytest.mark.gpu

WIDTHS = [1, 7, 8, 9, 16, 17, 33]
CASES = {  # kind, side, block: 8-dof levels of sides 8 and 2; 12, 6 (and 3); 6; 4
    "wilson_4": ("wilson2d", 32, 4, 3),
    "wilson_2": ("wilson2d", 24, 2, 4),
    "gauge_8": ("gauge2d", 48, 8, 2),
    "gauge_4": ("gauge2d", 16, 4, 3),
}


def _problem(name, precision, **kw):
    import paper_2108_11281_amd as m
    kind, N, blk, L = CASES[name]
    th = gauge_field(N, sigma=0.3, seed=4)
    A = operators.wilson2d(N, th, 0.2) if kind == "wilson2d" else operators.gauge_laplacian(N, th, 0.1)
    est = m.TraceEstimator(kind, N, L, L, mass=0.2 if kind == "wilson2d" else 0.1, field=th,
                           block=blk, n_vec=8, setup_sweeps=4, setup_seed=1, nb=max(WIDTHS),
                           precision=precision, nu_pre=1, nu_post=2, **kw)
    As, Ps, side, dof = [sp.csr_matrix(A)], [], N, 2 if kind == "wilson2d" else 1
    for l in range(L - 1):
        q = est.export_prolongation(l + 1, 8)
        y, x = np.divmod(np.arange(side * side), side)
        agg = np.repeat((y // blk) * (side // blk) + x // blk, dof)
        rows = np.repeat(np.arange(len(agg)), 8)
        P = sp.csr_matrix((q.ravel(), (rows, (agg[:, None] * 8 + np.arange(8)).ravel())))
        As.append((P.conj().T @ As[-1] @ P).tocsr())
        Ps.append(P)
        side, dof = side // blk, 8
    return est, As, Ps


def _random(rng, w, n):
    return rng.standard_normal((w, n)) + 1j * rng.standard_normal((w, n))


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("name", list(CASES))
def test_kernels_at_every_width(name, precision):
    require_gpu()
    est, A, P = _problem(name, precision)
    rng = np.random.default_rng(7)
    L = len(A)
    # FP64: sums of at most 128 products; FP32 sweeps: a few FP32 roundings per update
    tol = 1e-12
    for w in WIDTHS:
        for l in range(1, L):
            X = _random(rng, w, A[l].shape[0])
            ref = (A[l] @ X.T).T
            Y = from_dev(est.apply(l + 1, to_dev(X)), complex_=True)
            assert np.max(np.abs(Y - ref)) <= tol * np.max(np.abs(ref)), (w, l)
            Xf = _random(rng, w, A[l - 1].shape[0])
            ref = (P[l - 1].conj().T @ Xf.T).T
            Y = from_dev(est.restrict(l, to_dev(Xf)), complex_=True)
            assert np.max(np.abs(Y - ref)) <= tol * np.max(np.abs(ref)), (w, l)
            if l < L - 1:
                B = _random(rng, w, A[l].shape[0])
                colour = np.repeat(hierarchy.site_coloring(int(np.sqrt(A[l].shape[0] // 8))), 8)
                for reverse, zero in [(False, False), (True, False), (False, True)]:
                    Y = from_dev(est.smooth(l + 1, to_dev(B), None if zero else to_dev(X), 1,
                                            reverse, zero_start=zero), complex_=True)
                    for k in range(w):
                        ref = hierarchy.rbgs_sweeps(A[l], B[k], 0 * X[k] if zero else X[k], colour,
                                                    1, reverse)
                        assert np.max(np.abs(Y[k] - ref)) <= (
                            1e-11 if precision == "fp64" else 1e-5) * np.max(np.abs(ref)), (w, l, k)
    est.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("name", ["wilson_4", "wilson_2"])
def test_solve_of_an_8_dof_level(name, precision):
    require_gpu()
    # stopped early: the reported residuals are the residual kernel's partial sums
    est, A, _ = _problem(name, precision, krylov_restart=1, solve_tol=1e-2)
    rng = np.random.default_rng(8)
    for w in WIDTHS:
        b = _random(rng, w, A[1].shape[0])
        B, Y, rel = to_dev(b), est._vec(2, w), np.zeros(w)
        rc = est._lib.mlmc_solve(est._ctx, 2, w, ctypes.c_void_p(B.data_ptr()),
                                 ctypes.c_void_p(Y.data_ptr()),
                                 rel.ctypes.data_as(ctypes.POINTER(ctypes.c_double)))
        assert rc in (0, -4)
        r = b - (A[1] @ from_dev(Y, complex_=True).T).T
        ref = np.linalg.norm(r, axis=1) / np.linalg.norm(b, axis=1)
        # rounding of r: 1e-16 of A y against residuals above 1e-9
        assert np.all((ref > 1e-9) & (ref < 1e-1)), ref
        assert np.all(np.abs(rel - ref) <= 1e-6 * ref), w
    est.close()
