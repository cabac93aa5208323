"""Synthesis by waves of a few models: against the oracle at the edges of the
waves' shares, of the matrix product's columns and of the chunks of points;
the same bits whatever the number of models, with and without noise and
Jacobian, and the bits of the model-per-lane kernel, also for models whose
contributions overflow at some points only."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

vf = pytest.importorskip("paper_0901_2702_amd")

SPECS = {
    "hmi": wl.hmi_instrument,
    "wide": lambda: wl.hmi_instrument(n_fine=65, fwhm_mA=130.0),
    "fine": wl.fine_instrument,
    "band13": lambda: wl.fine_instrument(n_obs=13),  # 13 + 3 blocks: exactly one chunk
    "band14": lambda: wl.fine_instrument(n_obs=14),  # one row into the second chunk
    "band5": lambda: wl.fine_instrument(n_obs=5),
}
LANES_FROM = 114689  # HMI values without Jacobian: a model per lane


@pytest.fixture(scope="module")
def ctx():
    return vf.Context(0)


def _inst(ctx, spec):
    return vf.Instrument(ctx, spec.lambda0_A, spec.geff, spec.fine_offset_mA, spec.filter)


@pytest.mark.parametrize("name", sorted(SPECS))
def test_synthesis_at_the_edges(ctx, name):
    spec = SPECS[name]()
    inst = _inst(ctx, spec)
    oi = oracle.Instrument(spec.lambda0_A, spec.geff, spec.fine_offset_mA, spec.filter)
    n = 4 * 2048 + 5  # shares of 3 (values) and of 5 models (Jacobian), the last ones smaller
    P = wl.draw_params(n, 21).astype(np.float32)
    E = wl.draw_noise(n, spec.n_obs, 22).astype(np.float32)
    Pd, Ed = torch.from_numpy(P).to(ctx.device), torch.from_numpy(E).to(ctx.device)
    S, J = vf.synthesize(ctx, inst, Pd, jac=True)
    pick = np.r_[0:9, n - 7:n]
    ref = [oracle.forward(oi, P[k].astype(np.float64), jac=True) for k in pick]
    Sr, Jr = np.array([r[0] for r in ref]), np.array([r[1] for r in ref])
    assert np.max(np.abs(S[pick].cpu().numpy() - Sr)) < 2e-6
    colmax = np.abs(Jr).max(axis=(1, 2), keepdims=True)
    typical = np.median(np.abs(Jr).max(axis=(1, 2)), axis=0)
    assert (np.abs(J[pick].cpu().numpy() - Jr) <= 2e-4 * colmax + 3e-5 * typical).all()
    assert torch.equal(vf.synthesize(ctx, inst, Pd), S)
    for m in (1, 2, 3, 4, 5, 8, 9, 33, 2049, n):
        a = vf.synthesize(ctx, inst, Pd[n - m:])
        b, Jb = vf.synthesize(ctx, inst, Pd[n - m:], noise=Ed[n - m:], jac=True)
        c = vf.synthesize(ctx, inst, Pd[n - m:], noise=Ed[n - m:])
        assert torch.equal(a, S[n - m:]) and torch.equal(Jb, J[n - m:]), m
        assert torch.equal(b, S[n - m:] + Ed[n - m:]) and torch.equal(c, b), m


def test_models_that_overflow(ctx):
    spec = wl.hmi_instrument()
    inst = _inst(ctx, spec)
    P = wl.draw_params(LANES_FROM, 23).astype(np.float32)
    for k in range(0, 2000, 5):  # some overflow at the line's centre alone
        P[k, 5] = 10.0 ** (8 + k % 31)
        P[k, 4] = 1.0 + k % 7
    P[1, 3], P[2, 0], P[6, 7] = np.nan, np.inf, np.inf
    Pd = torch.from_numpy(P).to(ctx.device)
    lanes = vf.synthesize(ctx, inst, Pd)
    assert not torch.isfinite(lanes[:2000]).all()
    for m in (2000, 2003):
        a, b = vf.synthesize(ctx, inst, Pd[:m]), lanes[:m]
        c, _ = vf.synthesize(ctx, inst, Pd[:m], jac=True)
        for x in (a, c):
            assert ((x == b) | (x.isnan() & b.isnan())).all(), m
