"""The V-cycle of matrix-given operators rounds the same on every route: small levels as
one workgroup per vector for wide batches only (or for narrow ones too), a launch per
operation otherwise.  One preconditioned FP32 step of the same vectors in a narrow and
in a wide batch, bit for bit."""
import ctypes

import numpy as np
import pytest

from tests.gpu_util import from_dev, require_gpu, to_dev
from tests.test_gpu_rows import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["graph_inside", "graph_outside", "laplace_wide", "bilinear"])
def test_narrow_and_wide_batches_round_alike(name):
    require_gpu()
    import paper_2108_11281_amd as m
    A, L, kw = _problem(name)
    est = m.TraceEstimator("csr", 0, L, L, matrix=A, nb=66, precision="fp32_ir64", nu_pre=2,
                           nu_post=2, max_iter=1, max_refine=1, solve_tol=1e-14, **kw)
    b = np.random.default_rng(5).standard_normal((66, A.shape[0]))
    out = {}
    for w in (1, 9, 16, 17, 66):
        B, Y = to_dev(b[:w]), est._vec(1, w)
        rc = est._lib.mlmc_solve(est._ctx, 1, w, ctypes.c_void_p(B.data_ptr()),
                                 ctypes.c_void_p(Y.data_ptr()), None)
        assert rc in (0, -4)
        out[w] = from_dev(Y)
    for w in (1, 9, 16, 17):
        # the step length is a quotient of FP64 sums whose grouping may follow the width
        # (about 1e-16); its FP32 value, and with it the step, does not
        assert np.array_equal(out[w], out[66][:w]), w
    est.close()
