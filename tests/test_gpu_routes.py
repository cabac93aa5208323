"""Which kernel a call takes (csrc/routes.h).  Fits, seen in the waves that the
launch counted: the group inverter below its limit for the instrument's size, a
pixel per lane (a wave per 64 pixels) above it, with the same bits in both.
Re-fits, whose count only the device knows: the kernel that has nothing to do
ends at once and counts no waves.  Synthesis: the same bits on both sides of its
limits."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

vf = pytest.importorskip("paper_0901_2702_amd")
from paper_0901_2702_amd import learned  # noqa: E402

LANES = dict(chunk_log2=8)  # an explicit schedule: a pixel per lane


@pytest.fixture(scope="module")
def ctx():
    return vf.Context(0)


def _inputs(ctx, spec, n, seed):
    inst = vf.Instrument.from_spec(ctx, spec)
    P = torch.tensor(wl.draw_params(n, seed).astype(np.float32), device=ctx.device)
    noise = torch.tensor(wl.draw_noise(n, spec.n_obs, seed).astype(np.float32), device=ctx.device)
    return inst, vf.synthesize(ctx, inst, P, noise=noise), torch.tensor(wl.weights(spec.n_obs), device=ctx.device)


def _lanes(ctx, n):
    cus = torch.cuda.get_device_properties(ctx.device).multi_processor_count
    return min(4 * cus, (n + 63) // 64)


@pytest.mark.parametrize("name,spec,below,above,kw", [
    ("7 points", lambda: wl.hmi_instrument(n_fine=13), 8001, 20001, {}),
    ("29 points", lambda: wl.hmi_instrument(n_fine=51), 30001, 57001, {}),
    ("3 samples", lambda: wl.fine_instrument(n_obs=3), 16001, 40001, {}),
    ("14 samples", lambda: wl.fine_instrument(n_obs=14), 40001, 90001, {}),
    ("no trial", wl.hmi_instrument, 300, 3001, dict(max_iter=0)),
    ("five trials", wl.hmi_instrument, 15001, 60001, dict(max_iter=5)),
    ("19 points, three trials", lambda: wl.hmi_instrument(n_fine=33), 101, 2001, dict(max_iter=3)),
])
def test_small_instruments_and_short_fits(ctx, name, spec, below, above, kw):
    inst, o, W = _inputs(ctx, spec(), above, 61)
    print("[gpu] routes %s: lanes" % name, flush=True)
    ref = vf.invert(ctx, inst, o, W, opts=vf.Options(**LANES, **kw))
    assert ctx.counters()["grid_waves"] == _lanes(ctx, above)
    for n, lanes in ((above, True), (below, False)):
        print("[gpu] routes %s: %d pixels" % (name, n), flush=True)
        out = vf.invert(ctx, inst, o[:n], W, opts=vf.Options(**kw))
        assert (ctx.counters()["grid_waves"] == _lanes(ctx, n)) == lanes, n
        for k in ref:
            assert torch.equal(out[k], ref[k][:n]), (n, k)


def test_a_tuned_context_is_no_slower_than_an_untuned_one():
    """Tuned on its whole batch, a context keeps the group inverter where that
    is faster; tuned on a sample, it keeps the schedule for the size it was
    tuned for and no other."""
    for n, sample, lanes in ((24001, 0, ()), (30001, 4096, (30001, 36001))):
        ctx = vf.Context(0)
        inst, o, W = _inputs(ctx, wl.hmi_instrument(), 40001, 68)
        ref = vf.invert(ctx, inst, o, W)
        print("[gpu] routes: autotune on %d of %d" % (sample or n, n), flush=True)
        t = vf.autotune(ctx, inst, o[:n].contiguous(), W, sample=sample)
        print("[gpu] routes: %s" % t, flush=True)
        assert 0 < t["best_ms"] <= t["default_ms"] * 1.02
        for m in (5001, 16384, 24001, 30001, 36001, 40001):
            out = vf.invert(ctx, inst, o[:m], W)
            waves = ctx.counters()["grid_waves"]
            assert (waves == min(t["grid_waves"], (m + 63) // 64)) == (m in lanes), (n, m, waves)
            for k in ref:
                assert torch.equal(out[k], ref[k][:m]), (n, m, k)


@pytest.mark.parametrize("name,spec", [("HMI", wl.hmi_instrument), ("spectra", wl.fine_instrument)])
def test_derivative_passes_are_passes(ctx, name, spec):
    """The group inverter's trials run without derivatives; each accepted model
    that goes on has a derivative pass, a start has one pass for both."""
    inst, o, W = _inputs(ctx, spec(), 500, 67)
    print("[gpu] routes: passes of %s" % name, flush=True)
    vf.invert(ctx, inst, o, W)
    c = ctx.counters()
    assert c["derivative_passes"] == c["jacobians"]
    assert c["passes"] == c["trials"] + c["jacobians"] and c["jacobians"] > c["pixels"] == 500
    vf.invert(ctx, inst, o, W, opts=vf.Options(deriv_split=4))
    d = ctx.counters()
    for k in ("trials", "accepts", "jacobians"):
        assert d[k] == c[k], k
    assert d["derivative_passes"] >= c["derivative_passes"] and d["passes"] > d["derivative_passes"]


@pytest.mark.parametrize("n,refit,kernels", [
    (3000, False, ("group",)),
    (3000, True, ("group", "group")),
    (60001, False, ("lanes",)),          # above the short fit's limit, nothing to re-fit
    (60001, True, ("lanes", "lanes")),   # more re-fits than the group inverter takes
])
def test_learned_path_counts_the_waves_that_worked(ctx, n, refit, kernels):
    """An untrained network: every fit is above (refit) or below the threshold."""
    inst, o, W = _inputs(ctx, wl.hmi_instrument(), 3000, 65)
    o = o.repeat(21, 1, 1)[:n].contiguous()
    rng = np.random.default_rng(66)
    net = learned.Mlp(ctx, 24, rng.normal(size=24) * 0.01, np.full(24, 0.05),
                      np.array([0.0, 35.0, 0.25, 15.5, 0.3, 0.7, 0.6]),
                      np.array([1.7, 8.7, 0.14, 8.4, 0.12, 0.12, 0.23]), seed=1)
    tau = 1e-9 if refit else 1e30
    print("[gpu] routes learned n=%d refit=%s" % (n, refit), flush=True)
    ref = learned.invert_learned(ctx, inst, net, o, W, opts=vf.Options(**LANES), chi2_accept=tau)
    out = learned.invert_learned(ctx, inst, net, o, W, chi2_accept=tau)
    waves = ctx.counters()["grid_waves"]
    for k in ref:
        assert torch.equal(out[k], ref[k]), k
    assert int((out["status"] & vf.FALLBACK_USED).ne(0).sum()) == (n if refit else 0)
    cus = torch.cuda.get_device_properties(ctx.device).multi_processor_count
    group = waves // len(kernels)
    want = {"lanes": _lanes(ctx, n), "group": group}
    assert waves == sum(want[k] for k in kernels)
    if "group" in kernels:  # one or two full waves of it per SIMD
        assert group in (min(n, 4 * cus), min(n, 8 * cus))


def test_batches_left_to_the_lanes(ctx):
    """Wide spectra go to the group inverter, the other batches, together over
    their limits, to the lanes: two banded ones with their interleaved copies."""
    made = [_inputs(ctx, spec, n, 70 + i) for i, (spec, n) in enumerate(
        ((wl.fine_instrument(), 70), (wl.fine_instrument(n_obs=5), 40001),
         (wl.hmi_instrument(), 901), (wl.fine_instrument(n_obs=14), 20003)))]
    print("[gpu] routes: batches", flush=True)
    out = vf.invert_batches(ctx, [dict(inst=i, stokes=o, W=W) for i, o, W in made])
    waves = ctx.counters()["grid_waves"]
    assert waves == 70 + _lanes(ctx, 70 + 40001 + 901 + 20003)
    for (i, o, W), got in zip(made, out):
        alone = vf.invert(ctx, i, o, W, opts=vf.Options(**LANES))
        for k in alone:
            assert torch.equal(alone[k], got[k]), (i.n_obs, k)


@pytest.mark.parametrize("name,spec,sizes", [
    ("7 points", lambda: wl.hmi_instrument(n_fine=13), (5001, 7003, 20001)),
    ("29 points", lambda: wl.hmi_instrument(n_fine=51), (20001, 31003, 60001)),
    ("HMI", wl.hmi_instrument, (60001, 114689)),
    ("1 sample", lambda: wl.fine_instrument(n_obs=1), (8001, 12003, 20001)),
    ("5 samples", lambda: wl.fine_instrument(n_obs=5), (15001, 25003, 40001)),
    ("14 samples", lambda: wl.fine_instrument(n_obs=14), (15001, 25003, 40001)),
    ("20 samples", lambda: wl.fine_instrument(n_obs=20), (20001, 50003, 99001)),
])
def test_synthesis_on_both_sides(ctx, name, spec, sizes):
    spec = spec()
    inst = vf.Instrument.from_spec(ctx, spec)
    n = sizes[-1]
    P = wl.draw_params(n, 62).astype(np.float32)
    P[3, 5], P[40, 0], P[77, 7] = 1e30, np.inf, np.nan
    Pd = torch.tensor(P, device=ctx.device)
    E = torch.tensor(wl.draw_noise(n, spec.n_obs, 63).astype(np.float32), device=ctx.device)
    print("[gpu] routes synthesis %s" % name, flush=True)
    S, J = vf.synthesize(ctx, inst, Pd, jac=True)
    for m in sizes:
        a = vf.synthesize(ctx, inst, Pd[:m])
        b, Jb = vf.synthesize(ctx, inst, Pd[:m], noise=E[:m], jac=True)
        c = vf.synthesize(ctx, inst, Pd[:m], noise=E[:m])
        for x, y in ((a, S[:m]), (Jb, J[:m]), (b, S[:m] + E[:m]), (c, b)):
            assert torch.equal(torch.nan_to_num(x, nan=7e33), torch.nan_to_num(y, nan=7e33)), m


def test_more_models_than_a_launch_has_lanes_for(ctx):
    """1,074,790,400 models: at 16 models per wave of 64 lanes more than 2^32 lanes."""
    inst = vf.Instrument.from_spec(ctx, wl.fine_instrument(n_obs=1))
    base = torch.tensor(wl.draw_params(1 << 20, 64).astype(np.float32), device=ctx.device)
    print("[gpu] routes: 1025 x 2^20 models", flush=True)
    ref = vf.synthesize(ctx, inst, base)
    S = vf.synthesize(ctx, inst, base.repeat(1025, 1)).view(1025, 1 << 20, 4, 1)
    for k in (0, 511, 1023, 1024):
        assert torch.equal(S[k], ref), k
    del S
    torch.cuda.empty_cache()
