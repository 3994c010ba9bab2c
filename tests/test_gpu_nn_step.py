"""Loss and weight gradient of the learned smoother's network over numbers of crops at
the edges of the reduction's blocks (of 32 crops, of 512 for the loss) and of the kept
workspace."""
import numpy as np
import pytest

from oracle import nn
from tests.gpu_util import require_gpu
from tests.test_gpu_learned import bf16_round, cosine, rel_l2
from workloads import gauge_field, nn_init_weights

pytestmark = pytest.mark.gpu


def test_loss_and_gradient_over_crop_counts():
    require_gpu()
    import paper_2108_11281_amd as m
    import torch
    N = 32
    est = m.TraceEstimator("wilson2d", N, 2, 2, mass=0.1, field=gauge_field(N, seed=2), block=4,
                           n_vec=8, setup_sweeps=2, precision="fp32_ir64", nb=4)
    rng = np.random.default_rng(9)
    X = bf16_round(rng.standard_normal((3, 22, 22, 8)))
    T = rng.standard_normal((3, 16, 16, 4)).astype(np.float32)
    w = bf16_round(nn_init_weights(5) * 2.0)
    est.set_nn_weights(w)
    one = [nn.loss_and_grad(X[i:i + 1].transpose(0, 3, 1, 2).astype(np.float64),
                            T[i:i + 1].transpose(0, 3, 1, 2).astype(np.float64),
                            w.astype(np.float64)) for i in range(3)]
    for crops in (33, 1, 31, 32, 513, 1025, 512, 64):   # grown, shrunk, beyond the kept size
        pick = np.arange(crops) % 3
        loss, grad = est.nn_loss_grad(torch.tensor(X[pick], device="cuda"),
                                      torch.tensor(T[pick], device="cuda"))
        ref_loss = np.mean([one[i][0] for i in pick])
        ref_grad = np.mean([one[i][1] for i in pick], axis=0)
        # BF16 operands: a few 2^-8 relative, as for a single crop
        assert abs(loss - ref_loss) <= 1e-2 * ref_loss, crops
        assert rel_l2(grad, ref_grad) <= 2e-2, (crops, rel_l2(grad, ref_grad))
        assert cosine(grad, ref_grad) >= 0.999, crops
    est.close()
