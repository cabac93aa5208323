"""The first layer's weights of a training step are fetched four k-steps of 32
inputs ahead: widths that end before, at and after a turn of the four."""
import numpy as np
import pytest

import paper_0901_2702_amd as vf
from test_gpu_mlp import BF16_BOUND, _random_net, _unpack
from test_gpu_train import _batch, _oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in", [64, 96, 127, 128, 129, 160, 256, 260, 1248])
def test_gradient_at_the_turns(n_in):
    ctx = vf.Context(0)
    net, flat, mean, std = _random_net(ctx, n_in, 21)
    x, t, xd, td = _batch(ctx, n_in, 96, mean, std)
    print("[gpu] train widths: %d inputs" % n_in, flush=True)
    g, loss = net.gradient(xd, td)
    L, R, A = _oracle(flat, n_in, mean, std, x, t)
    assert loss.item() == pytest.approx(L, rel=1e-4)
    G = _unpack(g.cpu().numpy(), n_in)
    for k in R:
        assert np.all(np.abs(G[k] - R[k]) <= BF16_BOUND * A[k] + 1e-12 * np.abs(R[k]).max()), k
