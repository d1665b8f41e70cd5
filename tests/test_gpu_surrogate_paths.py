"""Training on batches at the edges of the kernels' tiles, slices and stages."""
import numpy as np
import pytest
import torch

from oracle import mlp
from paper_2311_16043_amd import Surrogate
from workloads import mlp_init

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


def _batch(n, seed):
    rng = np.random.default_rng(seed)
    x = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    d = rng.normal(size=(n, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    return x, d, rng.uniform(0, 1, n).astype(np.float32)


BOX = (np.full(3, -1.0, np.float32), np.full(3, 1.0, np.float32))


@pytest.mark.parametrize("n", [33, 513, 1025, 2047])
def test_gradient_matches_the_oracle(n):
    """Loss and gradient against the oracle with bfloat16 operands. The kernel rounds the
    same operands and differs where a value lies near a rounding edge or a ReLU's zero,
    so per layer it stays well within what bfloat16 itself changes (the oracle with
    operands rounded against the oracle with operands in binary64)."""
    w = mlp_init.he_uniform(21)
    x, d, T = _batch(n, n)
    net = Surrogate([-1, -1, -1], [1, 1, 1], init_weights=torch.from_numpy(w))
    loss, grad = net.loss_grad(torch.from_numpy(x), torch.from_numpy(d), torch.from_numpy(T))
    want_loss, want = mlp.loss_and_grad(w, x, d, T, *BOX)
    _, wide = mlp.loss_and_grad(w, x, d, T, *BOX, bf16_emulation=False)
    assert abs(float(loss) - want_loss) <= 1e-3 * abs(want_loss)
    got = grad.cpu().numpy().astype(np.float64)
    for (W, b), (Wr, br), (Ww, bw) in zip(mlp.unpack(got), mlp.unpack(want), mlp.unpack(wide)):
        for g, r, e in ((W, Wr, Ww), (b, br, bw)):
            assert np.linalg.norm(r) > 0
            assert np.linalg.norm(g - r) <= np.linalg.norm(r - e)


# the active sample first and last in its batch, tile of 16, block of 32, slice (of 96 at
# 1,025 samples, of 128 at 2,047) and stage of 64
@pytest.mark.parametrize("n,at", [(1, 0), (33, 32), (64, 63), (513, 31), (513, 512), (1025, 0), (1025, 63), (1025, 64),
                                  (1025, 95), (1025, 96), (1025, 1023), (1025, 1024), (2047, 127), (2047, 128),
                                  (2047, 2046)])
def test_one_sample_alone_has_a_gradient(n, at):
    """Where every other target is what the network says, and its second output is zero
    by its weights, the batch's gradient is 1 / n of that sample's own. The two round
    different multiples of the same values to bfloat16, each by up to 2^-9: the head's by
    2 2^-9 between them, and the values of four layers by less than 2^-9 of their 2-norm
    each, so they agree to 6 2^-9; a sample lost or taken twice is off by all of it."""
    w = mlp_init.he_uniform(22)
    W5, b5 = mlp.unpack(w)[-1]   # views into w
    W5[:, 1] = 0.0
    b5[1] = 0.0
    x, d, _ = _batch(n, 100 + n)
    net = Surrogate([-1, -1, -1], [1, 1, 1], init_weights=torch.from_numpy(w))
    x, d = torch.from_numpy(x), torch.from_numpy(d)
    T = net.infer_xd(x, d)[0].cpu()
    T[at] = 1.0 - T[at].round()
    grad = net.loss_grad(x, d, T)[1].double()
    alone = net.loss_grad(x[at:at + 1], d[at:at + 1], T[at:at + 1])[1].double() / n
    assert float(alone.norm()) > 0
    assert float((grad - alone).norm()) <= 6 * 2.0 ** -9 * float(alone.norm())
