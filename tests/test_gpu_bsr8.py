"""Levels with four or eight complex unknowns per site (matrix-core block kernels):
operator, sweeps, restriction, whole V-cycle steps and reported residuals at the edges of the column groups, on
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
CASES = {  # kind, side, block, levels, n_vec: block levels of sides 8, 2; 12, 6, 3; 6; 4; ..
    "wilson_4": ("wilson2d", 32, 4, 3, 8),
    "wilson_72": ("wilson2d", 48, 4, 3, 8),   # coarsest 72: half a chunk, an odd number of tiles
    "wilson_2": ("wilson2d", 24, 2, 4, 8),
    "wilson_3": ("wilson2d", 36, 3, 3, 4),
    "gauge_8": ("gauge2d", 48, 8, 2, 8),
    "gauge_4": ("gauge2d", 32, 4, 3, 4),
    "gauge_2": ("gauge2d", 16, 2, 3, 4),
}


def _problem(name, precision, pre=1, post=2, **kw):
    import paper_2108_11281_amd as m
    kind, N, blk, L, nv = CASES[name]
    th = gauge_field(N, sigma=0.3, seed=4)
    A = operators.wilson2d(N, th, 0.2) if kind == "wilson2d" else operators.gauge_laplacian(N, th, 0.1)
    est = m.TraceEstimator(kind, N, L, L, mass=0.2 if kind == "wilson2d" else 0.1, field=th,
                           block=blk, n_vec=nv, setup_sweeps=4, setup_seed=1, nb=70,
                           precision=precision, nu_pre=pre, nu_post=post, **kw)
    As, Ps, side, dof = [sp.csr_matrix(A)], [], N, 2 if kind == "wilson2d" else 1
    for l in range(L - 1):
        q = est.export_prolongation(l + 1, nv)
        y, x = np.divmod(np.arange(side * side), side)
        agg = np.repeat((y // blk) * (side // blk) + x // blk, dof)
        rows = np.repeat(np.arange(len(agg)), nv)
        P = sp.csr_matrix((q.ravel(), (rows, (agg[:, None] * nv + np.arange(nv)).ravel())))
        As.append((P.conj().T @ As[-1] @ P).tocsr())
        Ps.append(P)
        side, dof = side // blk, nv
    return est, As, Ps


def _random(rng, w, n):
    return rng.standard_normal((w, n)) + 1j * rng.standard_normal((w, n))


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("name", [c for c in CASES if c != "wilson_72"])
def test_kernels_at_every_width(name, precision):
    require_gpu()
    est, A, P = _problem(name, precision)
    rng = np.random.default_rng(7)
    L, nv = len(A), CASES[name][4]
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
                colour = np.repeat(hierarchy.site_coloring(int(np.sqrt(A[l].shape[0] // nv))), nv)
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


def _vcycle(A, P, dofs, l, b, pre, post, omega):
    if l == len(A) - 1:
        return np.linalg.solve(A[l].toarray(), b)
    colour = np.repeat(hierarchy.site_coloring(int(np.sqrt(A[l].shape[0] // dofs[l]))), dofs[l])
    X = np.zeros_like(b)
    for k in range(b.shape[1]):
        X[:, k] = hierarchy.rbgs_sweeps(A[l], b[:, k], X[:, k], colour, pre, False)
    X = X + omega * (P[l] @ _vcycle(A, P, dofs, l + 1, P[l].conj().T @ (b - A[l] @ X), pre, post,
                                    omega))
    for k in range(b.shape[1]):
        X[:, k] = hierarchy.rbgs_sweeps(A[l], b[:, k], X[:, k], colour, post, True)
    return X


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("name,top,pre,post", [
    ("wilson_4", 2, 1, 1), ("wilson_4", 2, 2, 0), ("wilson_72", 2, 1, 1), ("wilson_2", 2, 1, 2),
    ("wilson_2", 2, 0, 1), ("gauge_4", 2, 1, 1), ("gauge_2", 2, 2, 2),
    # from the fine lattice: its residual of one colour restricted directly (even blocks)
    ("wilson_4", 1, 2, 1), ("wilson_2", 1, 1, 1), ("wilson_3", 1, 1, 1), ("gauge_8", 1, 1, 1)])
def test_one_step_is_the_vcycle(name, top, pre, post, precision):
    require_gpu()
    omega = 1.0 if pre == post else 1.2
    est, A, P = _problem(name, precision, pre=pre, post=post, omega=omega, krylov_restart=1,
                         solve_tol=0.9999)
    widths = WIDTHS + ([64, 70] if name == "wilson_72" else [])
    rng = np.random.default_rng(11)
    l0 = top - 1
    dofs = [2 if name.startswith("wilson") else 1] + [CASES[name][4]] * (len(A) - 1)
    b = _random(rng, max(widths), A[l0].shape[0]).T
    z = _vcycle(A[l0:], P[l0:], dofs[l0:], 0, b, pre, post, omega)
    # one minimal-residual step along M b
    w = A[l0] @ z
    ref = (z * ((w.conj() * b).sum(0) / (w.conj() * w).sum(0))).T
    for width in widths:
        Y, _ = est.solve(top, to_dev(b.T[:width]))
        err = np.max(np.abs(from_dev(Y, complex_=True) - ref[:width]), axis=1)
        # FP64: rounding through the dense inverse; FP32: of some hundred operations
        tol = 1e-10 if precision == "fp64" else 1e-4
        assert np.all(err <= tol * np.max(np.abs(ref[:width]), axis=1)), (width, err)
    est.close()
