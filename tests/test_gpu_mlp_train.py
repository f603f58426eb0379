"""The training kernels at the sizes where their tiles end: gradients of ragged batches against
the FP64 reference with BF16 rounding, and an Adam step of every member against the published
update of its own gradient on the rows the documented hash draws."""
import numpy as np
import pytest

from oracle import mlp_oracle as M
from paper_1608_01125_amd import tril as T

from test_gpu_mlp import torch  # noqa: F401

pytestmark = pytest.mark.gpu


def _rows(n, seed):
    rng = np.random.default_rng(seed)
    x = rng.normal(0, 1, (n, 6)).astype(np.float32)
    y = (np.sin(x[:, 0]) + 0.3 * x[:, 1] * x[:, 2]).astype(np.float32)
    return x, y


@pytest.mark.parametrize("n", [1, 5, 63, 64, 65, 511, 545, 1056])
def test_gradient_of_ragged_batches(torch, n):  # noqa: F811
    """Each parameter block within 1e-3 of its norm (the full batch's bound; a BF16 rounding
    that falls the other way moves one of 256 activations by 2^-8, 2.4e-4 of a norm), four
    times that for batches of a few rows, where few elements share it."""
    x, y = _rows(n, n)
    net = T.Mlp(2, seed=4)
    try:
        loss, g = net.grad(1, torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
        p = net.get_params(1)
    finally:
        net.close()
    tol = 1e-3 if n >= 63 else 4e-3
    ref_loss, ref = M.loss_and_grad(p.astype(np.float64), x.astype(np.float64),
                                    y.astype(np.float64), np.zeros(6), np.ones(6), 0.0, 1.0, 256,
                                    bf16_points=True)
    assert abs(loss - ref_loss) <= tol * ref_loss
    off = 0
    for size in (1536, 256, 65536, 256, 65536, 256, 256, 1):
        a, b = g[off:off + size].astype(np.float64), ref[off:off + size]
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b) + 1e-12, (off, n)
        off += size


def _drawn(seed, k, step, n, batch):
    m = (1 << 64) - 1
    rows = []
    for i in range(batch):
        h = seed ^ (((k + 1) * 0x9E3779B97F4A7C15) & m) ^ ((step << 24) & m) ^ i
        for mul in (0xFF51AFD7ED558CCD, 0xC4CEB9FE1A85EC53):
            h = ((h ^ (h >> 33)) * mul) & m
        rows.append((h ^ (h >> 33)) % n)
    return np.array(rows)


@pytest.mark.parametrize("members,batch", [(1, 7), (3, 64), (2, 333)])
def test_first_adam_step_of_every_member(torch, members, batch):  # noqa: F811
    """w - lr g / (|g| + eps) (the first step's bias-corrected moments), the gradient of the
    drawn rows from tril_mlp_grad. Elements whose gradient is within rounding of zero may move
    either way and are left out; the others agree to FP32 rounding of w and of the update."""
    x, y = _rows(900, 3)
    lr = 1e-3
    net = T.Mlp(members, seed=8)
    try:
        before = [net.get_params(k).astype(np.float64) for k in range(members)]
        grads = []
        for k in range(members):
            r = _drawn(5, k, 0, len(x), batch)
            _, g = net.grad(k, torch.from_numpy(x[r]).cuda(), torch.from_numpy(y[r]).cuda())
            grads.append(g.astype(np.float64))
        net.train(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 1, batch, lr, 5)
        after = [net.get_params(k).astype(np.float64) for k in range(members)]
    finally:
        net.close()
    for w0, g, w1 in zip(before, grads, after):
        big = np.abs(g) > 1e-6
        ref = w0 - lr * g / (np.abs(g) + 1e-8)
        assert big.sum() > 1000
        tol = 2.0 ** -23 * np.abs(w0) + 1e-5 * lr
        assert np.all(np.abs(w1 - ref)[big] <= tol[big])
