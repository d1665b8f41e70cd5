"""Training on batches at the edges of the kernels' tiles, slices and stages."""
import numpy as np
import pytest
import torch

from paper_2311_16043_amd import Surrogate

from test_gpu_surrogate import test_grid_inference_with_fallback_matches_tracer as _check_fallback

pytestmark = pytest.mark.gpu


# tiles of 16 samples, blocks of 32, slices of a multiple of 32 in stages of 64 (1,025
# samples: slices of 96), 16 slices at most
@pytest.mark.parametrize("n", [1, 15, 31, 33, 64, 513, 1025, 2047])
def test_gradient_of_a_batch_taken_twice(n):
    """The mean loss over a batch and over the batch taken twice is the same, and
    halving every sample's gradient is exact in bfloat16, so the two gradients
    differ by the order of 2 n FP32 sums (a few n 2^-24 in the 2-norm)."""
    rng = np.random.default_rng(n)
    x = torch.from_numpy(rng.uniform(-1, 1, (n, 3)).astype(np.float32))
    d = rng.normal(size=(n, 3))
    d = torch.from_numpy((d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32))
    T = torch.from_numpy(rng.uniform(0, 1, n).astype(np.float32))
    net = Surrogate([-1, -1, -1], [1, 1, 1], seed=3)
    l1, g1 = net.loss_grad(x, d, T)
    l2, g2 = net.loss_grad(torch.cat([x, x]), torch.cat([d, d]), torch.cat([T, T]))
    assert abs(float(l1) - float(l2)) <= 1e-6 * abs(float(l1))
    assert torch.isfinite(g1).all() and float(g1.norm()) > 0
    assert float((g1.double() - g2.double()).norm() / g1.double().norm()) <= max(1e-5, 8 * n * 2.0 ** -24)


# the fallback list is dealt in chunks of 16 pools of 256 entries: less than a chunk, a
# round of chunks and one entry, and a list that is given more blocks (2.56M queries on)
@pytest.mark.parametrize("q0,qn,K", [(5, 3000, 32), (0, 2 * (8 * 16 * 256 + 1), 32), (0, 2_560_001, 160)])
def test_dealt_fallback_lists(q0, qn, K):
    _check_fallback(q0, qn, K)
