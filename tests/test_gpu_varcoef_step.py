"""The 3D V-cycle whole, one preconditioned step against a NumPy V-cycle: sides at the
edges of the plane march's row groups and segments (rows of 4 to 72 cells, one ragged
group of rows, one plane past a segment), the residual of one colour after the
pre-smoothing, odd numbers of columns, and no pre-smoothing (the full residual)."""
import ctypes

import numpy as np
import pytest

from oracle import hierarchy
from tests.gpu_util import from_dev, require_gpu, to_dev
from workloads import varcoef_faces

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 3, 9]


def _vcycle(A, P, sides, l, b, pre, post, omega):
    if l == len(A) - 1:
        return np.linalg.solve(A[l].toarray(), b)
    colour = hierarchy.site_coloring_3d(sides[l])
    d = A[l].diagonal()[:, None]
    classes = [np.flatnonzero(colour == c) for c in (0, 1)]
    rows = [A[l][c] for c in classes]
    x = np.zeros_like(b)

    def sweep(order):
        for c in order:   # within a class no cell couples to another
            i = classes[c]
            x[i] += (b[i] - rows[c] @ x) / d[i]

    for _ in range(pre):
        sweep((0, 1))
    x += omega * (P[l] @ _vcycle(A, P, sides, l + 1, P[l].T @ (b - A[l] @ x), pre, post, omega))
    for _ in range(post):
        sweep((1, 0))
    return x


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("N,L,pre,post", [(8, 3, 1, 1), (12, 2, 2, 1), (24, 3, 0, 1),
                                          (36, 3, 1, 2), (56, 4, 1, 1), (72, 4, 1, 1)])
def test_one_step_is_the_vcycle(N, L, pre, post, precision):
    require_gpu()
    import paper_2108_11281_amd as m
    faces = varcoef_faces(N, seed=7)
    A, P = hierarchy.varcoef_hierarchy(N, faces, 1e-2, L)
    omega = 1.2
    est = m.TraceEstimator("varcoef3d", N, L, L, shift=1e-2, field=faces, nb=max(WIDTHS),
                           precision=precision, nu_pre=pre, nu_post=post, omega=omega,
                           max_iter=1, max_refine=1, solve_tol=1e-14)
    rng = np.random.default_rng(3)
    b = rng.standard_normal((A[0].shape[0], max(WIDTHS)))
    z = _vcycle(A, P, [N >> l for l in range(L)], 0, b, pre, post, omega)
    ref = (z * ((b * z).sum(0) / (z * (A[0] @ z)).sum(0))).T
    for w in WIDTHS:
        B = to_dev(b.T[:w])
        Y = est._vec(1, w)
        rc = est._lib.mlmc_solve(est._ctx, 1, w, ctypes.c_void_p(B.data_ptr()),
                                 ctypes.c_void_p(Y.data_ptr()), None)
        assert rc in (0, -4)
        err = np.max(np.abs(from_dev(Y) - ref[:w]), axis=1) / np.max(np.abs(ref[:w]), axis=1)
        # FP64 rounding through the dense coarsest inverse; FP32: of some hundred
        # operations per unknown
        assert np.all(err <= (1e-11 if precision == "fp64" else 1e-4)), (w, err.max())
    est.close()
