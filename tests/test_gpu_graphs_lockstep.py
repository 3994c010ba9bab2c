"""HIP-graph replay where a solve still runs by launches: the refined CG of 2D Poisson
grids above side 128, whose iteration pairs have one graph after a refinement (the FP32
correction is written without reading it) and one otherwise, and of matrix-given operators
whose small levels are one launch inside the captured pair.  Replays are bitwise the
direct launches, in several solves with other work between them."""
import numpy as np
import pytest

from tests.gpu_util import from_dev, require_gpu, to_dev
from workloads import graph_laplacian

pytestmark = pytest.mark.gpu


def _compare(plain, graph, widths, level=1):
    import torch
    for rep in range(3):
        for w in widths:
            b = np.random.default_rng([rep, w]).standard_normal((w, plain.level_size(level)))
            Ya, ra = plain.solve(level, to_dev(b))
            ca = plain.counters()
            torch.zeros(1 << 20, device="cuda").sum().item()  # eager work between the replays
            Yb, rb = graph.solve(level, to_dev(b))
            cb = graph.counters()
            assert np.array_equal(from_dev(Ya), from_dev(Yb)) and np.array_equal(ra, rb), (rep, w)
            assert ca[:3] == cb[:3]
            yield ca
        for seed in (rep, rep + 7):
            assert np.array_equal(plain.sample_level(1, seed, 0, 21),
                                  graph.sample_level(1, seed, 0, 21))


@pytest.mark.parametrize("N,L", [(200, 3), (256, 4)])
def test_poisson_pairs_after_and_between_refinements(N, L):
    require_gpu()
    import paper_2108_11281_amd as m
    kw = dict(precision="fp32_ir64", nb=16, solve_tol=1e-13, inner_tol=1e-4, nu_pre=1, nu_post=1)
    plain = m.TraceEstimator("poisson2d", N, L, graphs=0, **kw)
    graph = m.TraceEstimator("poisson2d", N, L, graphs=1, **kw)
    for iterations, refinements, *_ in _compare(plain, graph, (1, 16)):
        pairs = (iterations - 2) // 2
        # both graphs: pairs that follow a refinement, more than once, and others
        assert refinements - 1 >= 2 and pairs > refinements - 1, (iterations, refinements)
    plain.close()
    graph.close()


@pytest.mark.parametrize("cycles", [1, 2])
def test_matrix_given_narrow_and_wide(cycles):
    require_gpu()
    import paper_2108_11281_amd as m
    kw = dict(matrix=graph_laplacian(20000), precision="fp32_ir64", nb=40, solve_tol=1e-11,
              omega=1.0, nu_pre=2, nu_post=2, top_cycles=cycles)
    plain = m.TraceEstimator("csr", 0, 3, 3, graphs=0, **kw)
    graph = m.TraceEstimator("csr", 0, 3, 3, graphs=1, **kw)
    for counts in _compare(plain, graph, (5, 40)):
        assert counts[0] >= 8  # the pair is replayed
    plain.close()
    graph.close()
