"""Products and transfers of a matrix-given operator on both sides of the batch size from
which a thread takes four vectors (2^19 rows x vectors), with vectors left over."""
import numpy as np
import pytest

from tests.gpu_util import from_dev, require_gpu, to_dev
from workloads import bilinear_prolongations, graph_laplacian, laplace_matrix

pytestmark = pytest.mark.gpu


def _close(got, M, x):
    """|got - M x| within the rounding of a row's sum, per entry"""
    ref, mag = (M @ x.T).T, (abs(M) @ abs(x).T).T
    k = np.diff(M.tocsr().indptr).max() + 2
    return np.all(np.abs(got - ref) <= k * np.finfo(float).eps * mag)


@pytest.mark.parametrize("name", ["graph", "bilinear"])
def test_products_and_transfers(name):
    require_gpu()
    import paper_2108_11281_amd as m
    if name == "graph":
        A, kw, widths = graph_laplacian(20000), {}, (1, 26, 27, 53, 54)
    else:
        A, kw = laplace_matrix(255), dict(prolongations=bilinear_prolongations(255, 4))
        widths = (1, 8, 9, 18, 19)
    n = A.shape[0]
    assert n * widths[1] < 1 << 19 <= n * widths[2]
    L = 4 if name == "bilinear" else 3
    est = m.TraceEstimator("csr", 0, L, L, matrix=A, nb=max(widths), precision="fp64", omega=1.0,
                           **kw)
    P = est.export_level(1, "P")
    rng = np.random.default_rng(2)
    for w in widths:
        x = rng.standard_normal((w, n))
        xc = rng.standard_normal((w, P.shape[1]))
        assert _close(from_dev(est.apply(1, to_dev(x))), A, x), w
        assert _close(from_dev(est.restrict(1, to_dev(x))), P.T.tocsr(), x), w
        assert _close(from_dev(est.prolong(1, to_dev(xc))), P, xc), w
    est.close()
