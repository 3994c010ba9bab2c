"""Sweeps of a matrix-given operator's small levels by themselves, one workgroup per
vector in the caller's blocks: the same bits as a launch per colour class and as shared
launches, at the edges of the lane groups, for every form of the call."""
import numpy as np
import pytest

from tests.gpu_util import from_dev, require_gpu, to_dev
from tests.test_gpu_rows import _problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32_ir64"])
@pytest.mark.parametrize("name", ["graph_inside", "laplace_wide", "bilinear"])
def test_schedules_give_the_same_bits(name, precision):
    require_gpu()
    import paper_2108_11281_amd as m
    A, L, kw = _problem(name)
    est = m.TraceEstimator("csr", 0, L, L, matrix=A, nb=66, precision=precision, omega=1.0, **kw)
    rng = np.random.default_rng(12)
    for level in range(1, L):
        n = est.level_size(level)
        for w in (1, 9, 66):
            b, x = (to_dev(rng.standard_normal((w, n))) for _ in range(2))
            forms = [dict(x=x, sweeps=s, reverse=r) for s in (1, 3) for r in (False, True)]
            forms += [dict(x=None, sweeps=2, zero_start=True), dict(x=x, sweeps=0),
                      dict(x=x, sweeps=2, restrict=True)]
            if 3 * 8 * n * w < 64 << 20:  # the fixed workspace
                forms.append(dict(x=x, sweeps=2, noalloc=True))
            for form in forms:
                form = dict(form)
                x0, sweeps = form.pop("x"), form.pop("sweeps")
                got = {s: est.smooth(level, b, x0, sweeps, schedule=s, **form)
                       for s in (None, "classes", "shared_tail")}
                parts = {s: [from_dev(t) for t in (y if isinstance(y, tuple) else (y,))]
                         for s, y in got.items()}
                for s in (None, "shared_tail"):
                    for p, q in zip(parts[s], parts["classes"]):
                        assert np.array_equal(p, q), (level, w, sweeps, form, s)
    est.close()
