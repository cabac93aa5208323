"""Damped systems whose factorisation breaks down at one pivot after the other
end in the eigen fallback, with the pseudo-inverse's step (singular values below
1e-12 of the largest discarded); systems with a tiny or a huge pivot, which it
leaves to plain divisions, keep the Cholesky step."""
import numpy as np
import pytest
import torch

import paper_0901_2702_amd as vf

pytestmark = pytest.mark.gpu
NPAR = 10


def _solve(full, g, eps):
    n = len(full)
    H = np.stack([full[:, p, q] for p in range(NPAR) for q in range(p + 1)], 1).astype(np.float32)
    ctx = vf.Context(0)
    print("[gpu] broken solve: %d systems" % n, flush=True)
    d, c = vf.solve(ctx, torch.from_numpy(H).to(ctx.device), torch.from_numpy(g).to(ctx.device),
                    torch.from_numpy(eps).to(ctx.device))
    return d.cpu().numpy(), c.cpu().numpy()


def test_breakdown_at_each_pivot():
    full = np.repeat(np.eye(NPAR)[None], 4 * NPAR, 0)
    eps = np.zeros(4 * NPAR)
    for j in range(NPAR):
        if j == 0:  # the first pivot is the damping alone
            eps[:4] = -1.0, -2.0, -1.5, -1.0
            continue
        # pivot j exactly zero, negative; twice with other pivots below one before it
        full[4 * j, j, j - 1] = 1.0
        full[4 * j + 1, j, j - 1] = 1.25
        full[4 * j + 2:4 * j + 4, 1:, 0] = 0.25
        full[4 * j + 2, j, 0] = 1.0
        full[4 * j + 3, j, 0] = 1.5
    g = np.random.default_rng(3).standard_normal((len(full), NPAR)).astype(np.float32)
    d, c = _solve(full, g, eps)
    assert (c == 1).all()
    for k, F in enumerate(full):
        low = np.tril(F)
        C = low + np.tril(low, -1).T + eps[k] * np.eye(NPAR)
        ref = np.linalg.pinv(C, rcond=1e-12, hermitian=True) @ g[k].astype(np.float64)
        assert np.abs(d[k] - ref).max() <= 1e-10 * np.abs(ref).max(), k


def test_pivots_out_of_the_quick_range_are_no_breakdown():
    full = np.repeat(np.eye(NPAR)[None], 3, 0)
    eps = np.array([0.0, 1e205, 1e250])
    g = np.ones((3, NPAR), np.float32)
    d, c = _solve(full, g, eps)
    assert (c == 0).all()
    assert np.allclose(d, (1.0 / (1.0 + eps))[:, None], rtol=1e-14, atol=0.0)
