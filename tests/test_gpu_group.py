"""The group inverter (a wave per pixel pass, for launches with fewer pixels
than lanes) against lm_kernel (a pixel per lane), which any explicit schedule
selects: the same bits for every per-pixel result and the same trials,
accepted trials and Jacobians, at the edges of its slots and chunks: one
pixel, fewer pixels than waves, more than all slots; a filter without
windowed records; banded spectra whose rows end inside, at and just past a
chunk of 16 rows; weights per pixel, starting models, frozen parameters, the
kept Hessian, no trial at all; non-finite pixels; normal equations that break
the Cholesky down; and the learned path, whose re-fit count only the device
knows and whose re-fits sum in lane pairs."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu

vf = pytest.importorskip("paper_0901_2702_amd")
from paper_0901_2702_amd import learned  # noqa: E402

LANES = dict(chunk_log2=8)  # an explicit schedule: lm_kernel


@pytest.fixture(scope="module")
def ctx():
    print("[gpu] group: creating context", flush=True)
    return vf.Context(0)


def _obs(spec, n, seed):
    oi = oracle.Instrument(spec.lambda0_A, spec.geff, spec.fine_offset_mA, spec.filter)
    P = wl.draw_params(n, seed)
    return (oracle.forward_batch(oi, P) + wl.draw_noise(n, spec.n_obs, seed)).astype(np.float32)


def _same(a, b, tag):
    for k in ("params", "chi2", "iters", "status"):
        x, y = a[k].cpu().numpy(), b[k].cpu().numpy()
        eq = (x == y) | (np.isnan(x) & np.isnan(y)) if x.dtype.kind == "f" else x == y
        assert np.all(eq), (tag, k, int(np.sum(~eq)))


def _both(ctx, inst, obs, W, tag, init=None, **kw):
    dev = ctx.device
    o, w = torch.tensor(obs, device=dev), torch.tensor(W, device=dev)
    i = None if init is None else torch.tensor(init, device=dev)
    print("[gpu] group %s: lanes" % (tag,), flush=True)
    ref = vf.invert(ctx, inst, o, w, init=i, opts=vf.Options(**LANES, **kw))
    torch.cuda.synchronize()
    cr = ctx.counters()
    print("[gpu] group %s: group" % (tag,), flush=True)
    out = vf.invert(ctx, inst, o, w, init=i, opts=vf.Options(**kw))
    torch.cuda.synchronize()
    c = ctx.counters()
    _same(ref, out, tag)
    for k in ("pixels", "trials", "accepts", "jacobians", "svd_fallbacks"):
        assert c[k] == cr[k], (tag, k)
    return out, c


SPECS = {
    "hmi": wl.hmi_instrument,                                     # windowed records
    "wide": lambda: wl.hmi_instrument(n_fine=65, fwhm_mA=130.0),  # six-row pass
    "fine": wl.fine_instrument,
    "band13": lambda: wl.fine_instrument(n_obs=13),  # 13 + 3 blocks: exactly one chunk
    "band14": lambda: wl.fine_instrument(n_obs=14),  # one row into the second chunk
    "band5": lambda: wl.fine_instrument(n_obs=5),
}


@pytest.mark.parametrize("name,n", [("hmi", 1), ("hmi", 5), ("hmi", 2049), ("hmi", 20011),
                                    ("wide", 300), ("fine", 1), ("fine", 3000), ("band5", 70),
                                    ("band13", 200), ("band14", 200)])
def test_group_gives_the_lane_results(ctx, name, n):
    spec = SPECS[name]()
    inst = vf.Instrument.from_spec(ctx, spec)
    _both(ctx, inst, _obs(spec, n, 31), wl.weights(spec.n_obs), (name, n))


@pytest.mark.parametrize("name", ["hmi", "fine"])
def test_options(ctx, name):
    spec = SPECS[name]()
    inst = vf.Instrument.from_spec(ctx, spec)
    n = 333
    obs = _obs(spec, n, 32)
    rng = np.random.default_rng(33)
    W = (wl.weights(spec.n_obs)[None] * rng.uniform(0.2, 2.0, (n, 4, spec.n_obs)))
    W[rng.random(W.shape) < 0.05] = 0.0
    W = W.astype(np.float32)
    init = wl.draw_params(n, 34).astype(np.float32)
    _both(ctx, inst, obs, W, (name, "weights, start, frozen"), init=init, free_mask=0x1FB)
    _both(ctx, inst, obs, W, (name, "kept Hessian"), hess_reuse=3.0)
    _both(ctx, inst, obs, W, (name, "no trial"), max_iter=0)
    W[::7] *= -1.0  # not served by the contract, and not different either
    _both(ctx, inst, obs, W, (name, "negative weights"))


@pytest.mark.parametrize("name", ["hmi", "fine"])
def test_pixels_that_cannot_be_fitted(ctx, name):
    spec = SPECS[name]()
    inst = vf.Instrument.from_spec(ctx, spec)
    obs = _obs(spec, 100, 35)
    W = np.ascontiguousarray(np.broadcast_to(wl.weights(spec.n_obs), obs.shape))
    obs[3, 0, 0] = np.nan
    obs[40, 3, spec.n_obs - 1] = np.inf
    W[77, 2, 1] = np.inf
    out, c = _both(ctx, inst, obs, W, (name, "non-finite"))
    st = out["status"].cpu().numpy()
    assert np.all(st[[3, 40, 77]] == vf.NONFINITE) and np.sum(st == vf.NONFINITE) == 3


def test_broken_down_systems(ctx):
    """Five weighted samples for ten parameters: J^T W J has rank five, and
    the Cholesky breaks down once the damping has become small."""
    spec = SPECS["hmi"]()
    inst = vf.Instrument.from_spec(ctx, spec)
    W = np.zeros((4, 6), np.float32)
    W[0, :5] = 1e6
    out, c = _both(ctx, inst, _obs(spec, 500, 36), W, "rank five", max_iter=200, rel_tol=0.0)
    print("[gpu] eigen fallbacks: %d" % c["svd_fallbacks"], flush=True)
    assert c["svd_fallbacks"] > 0


@pytest.mark.parametrize("name", ["hmi", "band14"])
def test_learned_path(ctx, name):
    """An untrained network: nearly every pixel is re-fitted."""
    spec = SPECS[name]()
    inst = vf.Instrument.from_spec(ctx, spec)
    n_in = 4 * spec.n_obs
    rng = np.random.default_rng(37)
    net = learned.Mlp(ctx, n_in, rng.normal(size=n_in) * 0.01, np.full(n_in, 0.05),
                      np.array([0.0, 35.0, 0.25, 15.5, 0.3, 0.7, 0.6]),
                      np.array([1.7, 8.7, 0.14, 8.4, 0.12, 0.12, 0.23]), seed=1)
    dev = ctx.device
    o = torch.tensor(_obs(spec, 3000, 38), device=dev)
    W = torch.tensor(wl.weights(spec.n_obs), device=dev)
    for tau in (0.0, 30.0):
        print("[gpu] group learned %s tau %g" % (name, tau), flush=True)
        ref = learned.invert_learned(ctx, inst, net, o, W, opts=vf.Options(**LANES),
                                     chi2_accept=tau)
        out = learned.invert_learned(ctx, inst, net, o, W, chi2_accept=tau)
        _same(ref, out, (name, tau))
        assert int((out["status"] & vf.FALLBACK_USED).ne(0).sum()) > 0


def test_batches(ctx):
    """Batches of both layouts, one of them empty, one with weights per pixel."""
    dev = ctx.device
    hs, fs = wl.hmi_instrument(), wl.fine_instrument()
    hi, fi = vf.Instrument.from_spec(ctx, hs), vf.Instrument.from_spec(ctx, fs)
    rng = np.random.default_rng(39)
    Wh = (wl.weights(6)[None] * rng.uniform(0.5, 1.5, (900, 4, 6))).astype(np.float32)
    batches = [dict(inst=fi, stokes=torch.tensor(_obs(fs, 300, 40), device=dev),
                    W=torch.tensor(wl.weights(fs.n_obs), device=dev)),
               dict(inst=hi, stokes=torch.zeros((0, 4, 6), device=dev),
                    W=torch.tensor(wl.weights(6), device=dev)),
               dict(inst=hi, stokes=torch.tensor(_obs(hs, 900, 41), device=dev),
                    W=torch.tensor(Wh, device=dev))]
    print("[gpu] group batches: lanes", flush=True)
    ref = vf.invert_batches(ctx, batches, opts=vf.Options(**LANES))
    cr = ctx.counters()
    print("[gpu] group batches: group", flush=True)
    out = vf.invert_batches(ctx, batches)
    c = ctx.counters()
    for i, (a, b) in enumerate(zip(ref, out)):
        _same(a, b, ("batches", i))
    for k in ("pixels", "trials", "accepts", "jacobians"):
        assert c[k] == cr[k], k


def test_batches_of_both_kernels(ctx):
    """More HMI pixels than the group inverter takes: they go to the lanes,
    the spectra of the same call to the group inverter."""
    dev = ctx.device
    hs, fs = wl.hmi_instrument(), wl.fine_instrument()
    hi, fi = vf.Instrument.from_spec(ctx, hs), vf.Instrument.from_spec(ctx, fs)
    obs = torch.tensor(_obs(hs, 2000, 42), device=dev).repeat(71, 1, 1).contiguous()
    batches = [dict(inst=hi, stokes=obs, W=torch.tensor(wl.weights(6), device=dev)),
               dict(inst=fi, stokes=torch.tensor(_obs(fs, 70, 43), device=dev),
                    W=torch.tensor(wl.weights(fs.n_obs), device=dev))]
    print("[gpu] group batches of both kernels", flush=True)
    ref = vf.invert_batches(ctx, batches, opts=vf.Options(**LANES))
    cr = ctx.counters()
    out = vf.invert_batches(ctx, batches)
    c = ctx.counters()
    for i, (a, b) in enumerate(zip(ref, out)):
        _same(a, b, ("both kernels", i))
    for k in ("pixels", "trials", "accepts", "jacobians"):
        assert c[k] == cr[k], k
