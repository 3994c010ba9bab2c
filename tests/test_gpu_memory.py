"""Device memory that an estimator holds."""
import gc

import pytest

from tests.gpu_util import require_gpu

pytestmark = pytest.mark.gpu


def test_small_coarsest_grids_hold_one_inverse():
    # a 64^2 coarsest grid is solved in the sine basis; of its explicit inverse (n^2 FP64
    # entries, 128 MiB) only the one that the exact coarsest trace and the export use
    torch = require_gpu()
    import paper_2108_11281_amd as m
    torch.zeros(1, device="cuda")
    gc.collect()  # estimators that earlier tests left
    before = torch.cuda.memory_allocated()
    est = m.TraceEstimator("poisson2d", 128, 2, nb=1, precision="fp32_ir64")
    held = torch.cuda.memory_allocated() - before
    inverse = 8 * est.level_size(2) ** 2
    assert inverse <= held <= inverse + (16 << 20)
    est.close()
