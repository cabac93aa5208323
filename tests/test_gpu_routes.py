"""Which kernel a fit takes (csrc/routes.h), seen in the waves that the launch
counted: the group inverter below its limit for the instrument's size, a pixel
per lane (a wave per 64 pixels) above it, with the same bits in both."""
import numpy as np
import pytest
import torch

import workloads as wl

pytestmark = pytest.mark.gpu

vf = pytest.importorskip("paper_0901_2702_amd")

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
    ("five trials", wl.hmi_instrument, 20001, 60001, dict(max_iter=5)),
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
