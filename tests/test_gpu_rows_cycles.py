"""Two coarse-grid cycles on the top level (top_cycles = 2) of matrix-given operators
whose levels one workgroup per vector runs alone: one preconditioned step against NumPy,
for narrow and wide batches."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import from_dev, require_gpu, to_dev
from tests.test_gpu_rows import _levels, _problem, _vcycle

pytestmark = pytest.mark.gpu


def _two_cycles(A, P, colour, b, pre, post, omega):
    M, d = A[0], A[0].diagonal()[:, None]
    classes = [np.flatnonzero(colour[0] == c) for c in range(colour[0].max() + 1)]
    x = np.zeros_like(b)
    for _ in range(pre):
        for c in classes:
            x[c] += (b[c] - M[c] @ x) / d[c]
    rc = P[0].T @ (b - M @ x)
    e = _vcycle(A, P, colour, 1, rc, pre, post, omega)
    if len(A) > 2:  # the coarsest level is solved exactly
        e = e + _vcycle(A, P, colour, 1, rc - A[1] @ e, pre, post, omega)
    x = x + omega * (P[0] @ e)
    for _ in range(post):
        for c in classes[::-1]:
            x[c] += (b[c] - M[c] @ x) / d[c]
    return x


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("name", ["graph_inside", "graph_outside", "laplace_wide", "bilinear"])
def test_one_step_has_both_cycles(name, precision):
    require_gpu()
    import paper_2108_11281_amd as m
    A, L, kw = _problem(name)
    pre, post, omega, widths = 1, 2, 1.0, (1, 16, 17, 66)
    est = m.TraceEstimator("csr", 0, L, L, matrix=A, nb=max(widths), precision=precision,
                           nu_pre=pre, nu_post=post, omega=omega, top_cycles=2, max_iter=1,
                           max_refine=1, solve_tol=1e-14, **kw)
    b = np.random.default_rng(6).standard_normal((A.shape[0], max(widths)))
    z = _two_cycles(*_levels(est, L, kw), b, pre, post, omega)
    # one CG iteration returns alpha M b with alpha = b^T M b / (M b)^T A (M b)
    ref = (z * ((b * z).sum(0) / (z * (A @ z)).sum(0))).T
    for w in widths:
        B, Y = to_dev(b.T[:w]), est._vec(1, w)
        rc = est._lib.mlmc_solve(est._ctx, 1, w, ctypes.c_void_p(B.data_ptr()),
                                 ctypes.c_void_p(Y.data_ptr()), None)
        assert rc in (0, -4)
        err = np.max(np.abs(from_dev(Y) - ref[:w]), axis=1) / np.max(np.abs(ref[:w]), axis=1)
        # as for one cycle: FP64 rounding of the dense coarsest inverse (condition below
        # 1e4), FP32 rounding of some hundred operations per unknown
        assert np.all(err <= (1e-11 if precision == "fp64" else 1e-4)), (w, err.max())
    est.close()
