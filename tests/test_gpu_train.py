"""The training step's row and gradient kernels at the edges of their shares:
batches of one workgroup's rows up to several, batch chunks that are empty or
end inside, input widths of one k-step and more, and workgroups of 32 rows
(from 131,072 on) against those of 16."""
import numpy as np
import pytest
import torch

from oracle import mlp as omlp
from test_gpu_mlp import BF16_BOUND, _abs_backward, _random_net, _unpack

pytestmark = pytest.mark.gpu

vf = pytest.importorskip("paper_0901_2702_amd")


@pytest.fixture(scope="module")
def ctx():
    return vf.Context(0)


def _batch(ctx, n_in, n, mean, std):
    rng = np.random.default_rng(n)
    x = (rng.normal(size=(n, n_in)) * std + mean).astype(np.float32)
    t = rng.normal(size=(n, 10)).astype(np.float32)
    return x, t, torch.tensor(x, device=ctx.device), torch.tensor(t, device=ctx.device)


def _oracle(flat, n_in, mean, std, x, t):
    P = _unpack(flat, n_in)
    xs = ((x - mean.astype(np.float32)) * (1.0 / std.astype(np.float32))).astype(np.float32)
    y, cache = omlp.forward(P, xs, emulate_bf16=True)
    return (np.sum((y - t) ** 2), omlp.backward(P, cache, t.astype(np.float64), emulate_bf16=True),
            _abs_backward(P, cache, t.astype(np.float64)))


@pytest.mark.parametrize("n_in,n", [(24, 32), (32, 544), (33, 96), (100, 160), (24, 4128)])
def test_gradient_at_the_edges(ctx, n_in, n):
    net, flat, mean, std = _random_net(ctx, n_in, 11)
    x, t, xd, td = _batch(ctx, n_in, n, mean, std)
    g, loss = net.gradient(xd, td)
    L, R, A = _oracle(flat, n_in, mean, std, x, t)
    assert loss.item() == pytest.approx(L, rel=1e-4)
    G = _unpack(g.cpu().numpy(), n_in)
    for k in R:
        assert np.all(np.abs(G[k] - R[k]) <= BF16_BOUND * A[k] + 1e-12 * np.abs(R[k]).max()), k


def test_workgroups_of_32_rows(ctx):
    """32 copies of 4,096 rows: every row's values are the same (the mean's
    1 / 32 is exact), so the loss is 32 times the block's and the gradients
    differ by the roundings of the longer sums alone."""
    net, flat, mean, std = _random_net(ctx, 24, 12)
    x, t, xd, td = _batch(ctx, 24, 4096, mean, std)
    g, loss = net.gradient(xd, td)
    G, LOSS = net.gradient(xd.repeat(32, 1).contiguous(), td.repeat(32, 1).contiguous())
    assert LOSS.item() == 32.0 * loss.item()
    a, b = _unpack(g.cpu().numpy(), 24), _unpack(G.cpu().numpy(), 24)
    _, _, A = _oracle(flat, 24, mean, std, x, t)
    for k in A:  # sums of 131,072 / 16 and of 4,096 / 16 terms in float32, then 16 of those
        assert np.all(np.abs(a[k] - b[k]) <= (8192 + 256 + 32) * 2.0 ** -24 * A[k]), k
