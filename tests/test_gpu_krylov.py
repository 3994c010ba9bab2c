"""The flexible GMRES of complex operators over restart lengths and sizes at which its
orthogonalisation changes route: dot products summed by the update itself (up to 64
blocks: 65536 unknowns) or by a launch between, one or four elements per thread."""
import numpy as np
import pytest

from tests.gpu_util import from_dev, require_gpu, to_dev
from workloads import gauge_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("restart", [1, 2, 4, 5, 16, 17, 32])
@pytest.mark.parametrize("N,widths", [(32, [1, 5, 9]), (192, [1, 4, 5])])
def test_solves_over_restarts(N, widths, restart, precision):
    require_gpu()
    import paper_2108_11281_amd as m
    est = m.TraceEstimator("wilson2d", N, 3, 3, mass=0.3, field=gauge_field(N, seed=5), block=4,
                           n_vec=4, setup_sweeps=4, nb=max(widths), precision=precision,
                           krylov_restart=restart, solve_tol=1e-10, max_refine=50)
    rng = np.random.default_rng(restart)
    n = est.level_size(1)
    for w in widths:
        b = rng.standard_normal((w, n)) + 1j * rng.standard_normal((w, n))
        b[w // 2] *= 1e-3
        Y, rel = est.solve(1, to_dev(b))
        assert np.all(rel <= 1e-10)
        r = b - from_dev(est.apply(1, Y), complex_=True)
        true = np.linalg.norm(r, axis=1) / np.linalg.norm(b, axis=1)
        # the reported residual is the true one up to FP64 rounding of A y
        assert np.all(np.abs(true - rel) <= 1e-13), (w, true, rel)
    est.close()


@pytest.mark.parametrize("N,width", [(32, 3), (192, 5)])
def test_one_cycle_is_the_minimal_residual(N, width):
    # a cycle of m steps in FP64 without a coarse level's help to hide an error: its
    # residual norm is no larger than after m - 1 steps, and strictly decreasing here
    require_gpu()
    import paper_2108_11281_amd as m
    th = gauge_field(N, seed=6)
    rng = np.random.default_rng(1)
    b = None
    last = None
    for restart in (1, 2, 3, 6, 12):
        est = m.TraceEstimator("wilson2d", N, 2, 2, mass=0.3, field=th, block=4, n_vec=4,
                               setup_sweeps=4, nb=width, precision="fp64",
                               krylov_restart=restart, solve_tol=0.5)
        if b is None:
            n = est.level_size(1)
            b = rng.standard_normal((width, n)) + 1j * rng.standard_normal((width, n))
        Y, rel = est.solve(1, to_dev(b))   # stops after the first cycle below 0.5
        r = b - from_dev(est.apply(1, Y), complex_=True)
        true = np.linalg.norm(r, axis=1) / np.linalg.norm(b, axis=1)
        assert np.all(true < 0.5)
        if last is not None:
            assert np.all(true < last + 1e-13), (restart, true, last)
        last = true
        est.close()
