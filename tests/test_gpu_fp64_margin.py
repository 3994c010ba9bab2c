"""Plain FP64 solves at tolerances near the rounding of their residuals, where the CG
recursion passes columns whose true residual misses: every column meets solve_tol, on
the grids that one workgroup per column solves and on the lockstep ones, for matrix-given
operators and for narrow FP64 batches of the FP32 mode."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import from_dev, require_gpu, to_dev
from workloads import graph_laplacian, laplace_matrix

pytestmark = pytest.mark.gpu

CASES = [("poisson", 64, 3, 2e-14), ("poisson", 128, 4, 5e-14), ("poisson", 256, 5, 1e-13),
         ("narrow", 256, 5, 1e-13), ("graph", 3000, 3, 5e-14)]


@pytest.mark.parametrize("name,N,L,tol", CASES)
def test_every_column_meets_the_tolerance(name, N, L, tol):
    require_gpu()
    import paper_2108_11281_amd as m
    w = 128
    if name == "graph":
        A = graph_laplacian(N)
        est = m.TraceEstimator("csr", 0, L, L, matrix=A, omega=1.0, nb=w, precision="fp64",
                               solve_tol=tol)
    else:
        A = laplace_matrix(N)
        kw = dict(precision="fp64") if name == "poisson" else \
            dict(precision="fp32_ir64", narrow_fp64=w)
        est = m.TraceEstimator("poisson2d", N, L, nb=w, solve_tol=tol, **kw)
    rng = np.random.default_rng(1)
    for _ in range(3):
        b = rng.standard_normal((w, A.shape[0]))
        B, Y, rel = to_dev(b), est._vec(1, w), np.zeros(w)
        rc = est._lib.mlmc_solve(est._ctx, 1, w, ctypes.c_void_p(B.data_ptr()),
                                 ctypes.c_void_p(Y.data_ptr()),
                                 rel.ctypes.data_as(ctypes.POINTER(ctypes.c_double)))
        assert rc == 0 and np.all(rel <= tol), (rc, int((rel > tol).sum()))
        y = from_dev(Y)
        res = np.linalg.norm(b - (A @ y.T).T, axis=1) / np.linalg.norm(b, axis=1)
        # the residual as formed here, with its own rounding of ten operations per entry
        fuzz = 10 * np.finfo(float).eps * np.linalg.norm(abs(A) @ abs(y.T), axis=0) / \
            np.linalg.norm(b, axis=1)
        assert np.all(res <= tol + fuzz)
    est.close()
