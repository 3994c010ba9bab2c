"""Plain FP64 solves of narrow batches in the FP32 mode (narrow_fp64) of matrix-given
operators: the route and the bits of the FP64 mode's solves, with small levels that one
workgroup per vector runs."""
import numpy as np
import pytest

from tests.gpu_util import from_dev, require_gpu, to_dev
from tests.test_gpu_rows import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["graph_inside", "graph_outside", "laplace_wide", "bilinear"])
def test_narrow_batches_are_the_fp64_solves(name):
    require_gpu()
    import paper_2108_11281_amd as m
    A, L, kw = _problem(name)
    common = dict(matrix=A, nb=32, nu_pre=1, nu_post=1, omega=1.0, solve_tol=1e-10, **kw)
    mixed = m.TraceEstimator("csr", 0, L, L, precision="fp32_ir64", narrow_fp64=20, **common)
    plain = m.TraceEstimator("csr", 0, L, L, precision="fp64", **common)
    b = np.random.default_rng(8).standard_normal((20, A.shape[0]))
    for w in (1, 8, 16, 17, 20):
        Y, rel = mixed.solve(1, to_dev(b[:w]))
        launches = {}
        for est in (mixed, plain):
            est.set_timing(["rbgs_sweep"])
            est.reset_kernel_stats()
            Z, _ = est.solve(1, to_dev(b[:w]))
            launches[est] = est.kernel_stats("rbgs_sweep", fp64=True)[0]
            est.set_timing(False)
        assert np.all(rel <= 1e-10)
        assert np.array_equal(from_dev(Y), from_dev(Z)), w
        # the same kernels: no level falls back to a launch per colour class
        assert launches[mixed] == launches[plain] > 0, w
    mixed.close()
    plain.close()
