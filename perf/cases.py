"""Performance cases: the calls that a user of the inverter makes, over the sizes they are made at.

A case is a dict of plain values.  `prepare` builds what a program holds before the call (context,
instrument, observed profiles, weights, a trained network), `run` is one pass through the public entry
points, `work` is what that pass cannot do without and `exact` is its result in 64 bits where it has one.

Observations are drawn from the synthetic priors (B 0-3000 G, isotropic inclination, ...) and synthesised
here in float64 with plain torch operations, plus N(0, 1e-3) noise, so that the inputs do not depend on the
library.  An inversion's result has no 64-bit value (a fit stops where its own rounding lets it), so `exact`
covers the synthesis, the starting models, the weights and the network.
"""
import math

import numpy as np
import torch

import paper_0901_2702_amd as vf
from paper_0901_2702_amd import learned

DEV = "cuda:0"
SIGMA = 1e-3
DEFAULT_MODEL = (1500.0, 90.0, 90.0, 0.0, 35.0, 0.25, 15.5, 0.3, 0.7, 0.6)


def listed():
    return [
        # a few pixels looked at by hand, each with weights of its own
        dict(name="hmi_pixels", kind="invert", inst="hmi", n=37, wpp=True),
        # a 64 x 64 cut-out of HMI filtergrams
        dict(name="hmi_64x64", kind="invert", inst="hmi", n=4096, wpp=False),
        # a 512 x 512 region, whole plain-LM call from the default model
        dict(name="hmi_512x512", kind="invert", inst="hmi", n=262144, wpp=False),
        # one slit position of a spectrograph: 112-sample spectra
        dict(name="fine_slit", kind="invert", inst="fine", n=1000, wpp=False),
        # a raster of slit positions
        dict(name="fine_raster", kind="invert", inst="fine", n=100003, wpp=False),
        # fine spectra and filtergrams together in one launch
        dict(name="mixed_batches", kind="batches", n=20000, n2=50001),
        # the benchmark's step: a million held-out pixels from the network's starts
        dict(name="learned_1M", kind="learned", n=1000000),
        # the same path at the size of one request to a service
        dict(name="learned_request", kind="learned", n=20011),
        # synthesis with the Jacobian (response of the filtergrams to the model)
        dict(name="synth_jacobian", kind="synth", inst="hmi", n=65537, jac=True, noise=False),
        # noisy spectra, as a training set is made
        dict(name="synth_spectra", kind="synth", inst="fine", n=30011, jac=False, noise=True),
        # one epoch of the initialiser's training
        dict(name="train_epoch", kind="train", n=262144, batch=4096),
        # classical starting models and per-pixel weights of an image strip
        dict(name="classical_weights", kind="classical", n=1000003),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("invert", "invert", "invert_fine", "batches", "learned", "synth", "train", "classical"))
    if kind == "invert":
        return dict(kind="invert", inst="hmi", n=_log_int(rng, 1, 262144), wpp=rng.random() < 0.5)
    if kind == "invert_fine":
        return dict(kind="invert", inst="fine", n=_log_int(rng, 1, 100003), wpp=rng.random() < 0.25)
    if kind == "batches":
        return dict(kind="batches", n=_log_int(rng, 64, 20000), n2=_log_int(rng, 64, 50001))
    if kind == "learned":
        return dict(kind="learned", n=_log_int(rng, 256, 1000000))
    if kind == "synth":
        inst = rng.choice(("hmi", "fine"))
        jac = rng.random() < 0.5
        return dict(kind="synth", inst=inst, n=_log_int(rng, 16, 65537 if inst == "hmi" else 30011), jac=jac,
                    noise=not jac)
    if kind == "train":
        batch = rng.choice((1024, 2048, 4096))
        return dict(kind="train", n=batch * rng.randint(8, 262144 // batch) + rng.randint(0, 999), batch=batch)
    return dict(kind="classical", n=_log_int(rng, 100, 1000003))


# ---- instruments -----------------------------------------------------------------------------------------
# hmi: Fe I 6173 A seen through six Gaussian filters; fine: Fe I 6302.5 A, 112 samples at 21.5 mA.

def _hmi_spec():
    fine = np.linspace(-600.0, 600.0, 101)
    sig = 76.0 / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    centres = np.array((-172.0, -103.2, -34.4, 34.4, 103.2, 172.0))
    filt = np.exp(-0.5 * ((fine[None, :] - centres[:, None]) / sig) ** 2)
    return 6173.3356, 2.5, fine, filt / filt.sum(axis=1, keepdims=True)


def _fine_spec():
    n_obs, step, over, pad, half = 112, 21.5, 4, 8, 7
    obs = (np.arange(n_obs) - (n_obs - 1) / 2.0) * step
    n_fine = n_obs * over + 2 * pad
    fine = obs[0] + (np.arange(n_fine) - pad) * (step / over)
    sig = 25.0 / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    filt = np.zeros((n_obs, n_fine))
    for j in range(n_obs):
        ks = np.arange(pad + over * j - half, pad + over * j + half + 1)
        w = np.exp(-0.5 * ((fine[ks] - obs[j]) / sig) ** 2)
        filt[j, ks] = w / w.sum()
    return 6302.4936, 2.5, fine, filt


_SPECS = {"hmi": _hmi_spec, "fine": _fine_spec}
_N_OBS = {"hmi": 6, "fine": 112}
_KEPT = {}


def _once(key, make):
    """What a program makes once and keeps: its context, instruments and network."""
    if key not in _KEPT:
        _KEPT[key] = make()
    return _KEPT[key]


def _ctx():
    return _once("ctx", lambda: vf.Context(0))


def _inst(name):
    return _once(("inst", name), lambda: vf.Instrument(_ctx(), *_SPECS[name]()))


# ---- 64-bit Milne-Eddington synthesis in torch ------------------------------------------------------------

def _weideman(N=32):
    L, M = math.sqrt(N / math.sqrt(2.0)), 8 * N
    th = np.arange(-M + 1, M) * math.pi / M
    t = L * np.tan(0.5 * th)
    f = np.exp(-t * t) * (L * L + t * t)
    return L, [float((f * np.cos(n * th)).sum() / (2.0 * M)) for n in range(N + 1)]


def _faddeeva(u, a):
    """Re and Im of w(u + i a) by the 32-term rational series of Weideman (1994)."""
    L, c = _once("weideman", _weideman)
    dr, di = L + a, -u
    den = dr * dr + di * di
    ir, ii = dr / den, -di / den
    zr, zi = (L * L - a * a - u * u) / den, 2.0 * L * u / den
    r, s = 2.0 * zr, zr * zr + zi * zi
    b2 = torch.full_like(u, c[32])
    b1 = c[31] + r * b2
    for k in range(30, 1, -1):
        b1, b2 = c[k] + r * b1 - s * b2, b1
    pr, pi = 2.0 * (b1 * zr + c[1] - s * b2), 2.0 * b1 * zi
    qr, qi = pr * ir - pi * ii + 1.0 / math.sqrt(math.pi), pr * ii + pi * ir
    return ir * qr - ii * qi, ir * qi + ii * qr


def _forward(spec, P):
    """Filtered Stokes vector [n, 4, n_obs] (float64) of the models P [n, 10]."""
    lam0, geff, fine, filt = spec
    x = torch.as_tensor(fine, device=P.device)[None, :]
    F = torch.as_tensor(filt, device=P.device).t().contiguous()
    B, g, psi, v, dl, a, eta, S0, S1, al = (P[:, q:q + 1] for q in range(10))
    g, psi = torch.deg2rad(g), torch.deg2rad(psi)
    up = (x - lam0 * 1000.0 * v / 299792.458) / dl
    zs = 4.66685e-10 * geff * lam0 * lam0 * B / dl
    a = a.expand_as(up)
    (Hp, Fp), (Hb, Fb), (Hr, Fr) = _faddeeva(up, a), _faddeeva(up + zs, a), _faddeeva(up - zs, a)
    s2, cg = torch.sin(g) ** 2, torch.cos(g)
    eI = 1.0 + 0.5 * eta * (Hp * s2 + 0.5 * (Hb + Hr) * (1.0 + cg * cg))
    eQ, rQ = (0.5 * eta * s2 * (p - 0.5 * (b + r)) for p, b, r in ((Hp, Hb, Hr), (Fp, Fb, Fr)))
    eV, rV = 0.5 * eta * cg * (Hr - Hb), 0.5 * eta * cg * (Fr - Fb)
    Pi, R2 = eQ * rQ + eV * rV, rQ * rQ + rV * rV
    D = eI * eI * (eI * eI - eQ * eQ - eV * eV + R2) - Pi * Pi
    I = al * eI * (eI * eI + R2) / D + (1.0 - al) / (1.0 + eta * Hp)
    Q, U, V = (-al * n / D for n in (eI * eI * eQ + rQ * Pi, eI * (eQ * rV - eV * rQ), eI * eI * eV + rV * Pi))
    I, Q, U, V = (t @ F for t in (I, Q, U, V))
    c2, s2p = torch.cos(2.0 * psi), torch.sin(2.0 * psi)
    return torch.stack((S0 * F.sum(0) + S1 * I, S1 * (c2 * Q - s2p * U), S1 * (s2p * Q + c2 * U), S1 * V), 1)


def _chunks(f, n, step):
    return torch.cat([f(i, min(n, i + step)) for i in range(0, n, step)])


def _draw_models(n, gen):
    """Models [n, 10] float32 from the synthetic priors."""
    r = torch.rand((10, n), generator=gen, device=DEV, dtype=torch.float64)
    lo = torch.tensor((0, 0, 0, -3, 20, 0, 1, 0.1, 0, 0.2), device=DEV, dtype=torch.float64)[:, None]
    hi = torch.tensor((3000, 0, 180, 3, 50, 0.5, 30, 0.5, 0, 1), device=DEV, dtype=torch.float64)[:, None]
    P = lo + r * (hi - lo)
    P[1] = torch.rad2deg(torch.arccos(2.0 * r[1] - 1.0))
    P[8] = 1.0 - P[7]
    return P.t().float().contiguous()


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) % (1 << 62))


def _observe(inst, n, gen):
    """Models and noisy observed profiles [n, 4, n_obs], float32."""
    P = _draw_models(n, gen)
    step = 65536 if inst == "hmi" else 16384
    S = _chunks(lambda i, j: _forward(_SPECS[inst](), P[i:j].double()).float(), n, step)
    return P, S + SIGMA * torch.randn(S.shape, generator=gen, device=DEV)


def _weights(inst, n, wpp, gen):
    shape = (n, 4, _N_OBS[inst]) if wpp else (4, _N_OBS[inst])
    W = torch.full(shape, SIGMA ** -2, device=DEV)
    return W * (0.25 + torch.rand(shape, generator=gen, device=DEV)) if wpp else W


# ---- the network ------------------------------------------------------------------------------------------

def _codes(P, mean, std):
    g, p2, b = torch.deg2rad(P[:, 1]), torch.deg2rad(2.0 * P[:, 2]), P[:, 0] / 3000.0
    B = torch.stack((b * torch.cos(g), b * torch.sin(g) * torch.cos(p2), b * torch.sin(g) * torch.sin(p2)), 1)
    return torch.cat((B, (P[:, 3:] - mean) / std), 1)


def _train_torch(steps=8000, batch=8192, pool=1500000):
    """Normalisation and packed weights of a network for the HMI filtergrams, trained with plain torch."""
    gen = _gen(77)
    P, S = _observe("hmi", pool, gen)
    X = S.reshape(pool, 24)
    mean, std, om, osd = X.mean(0), X.std(0), P[:, 3:].mean(0), P[:, 3:].std(0)
    X, T = (X - mean) / std, _codes(P, om, osd)
    was = torch.are_deterministic_algorithms_enabled()
    torch.use_deterministic_algorithms(True)
    try:
        dims = ((24, 256), (256, 256), (256, 256), (256, 10))
        ps = []
        for k, (i, o) in enumerate(dims):
            w = torch.randn((i, o), generator=gen, device=DEV) * math.sqrt((1.0 if k == 3 else 2.0) / i)
            ps += [w.requires_grad_(), torch.zeros(o, device=DEV, requires_grad=True)]
        opt = torch.optim.Adam(ps, lr=3e-3, fused=True)
        for t in range(steps):
            opt.param_groups[0]["lr"] = 3e-3 * (0.02 + 0.98 * 0.5 * (1.0 + math.cos(math.pi * t / steps)))
            at = (t * batch) % (pool - batch + 1)
            h = X[at:at + batch]
            for k in range(4):
                h = torch.addmm(ps[2 * k + 1], h, ps[2 * k])
                h = torch.nn.functional.gelu(h) if k < 3 else h
            opt.zero_grad(set_to_none=True)
            torch.nn.functional.mse_loss(h, T[at:at + batch]).backward()
            opt.step()
    finally:
        torch.use_deterministic_algorithms(was)
    pack = []
    for k, (i, o) in enumerate(dims):  # rows padded to 32 inputs, the last layer to 32 outputs
        w = torch.zeros((max(i, 32), max(o, 32)), device=DEV)
        w[:i, :o] = ps[2 * k].detach()
        b = torch.zeros(max(o, 32), device=DEV)
        b[:o] = ps[2 * k + 1].detach()
        pack += [w.reshape(-1), b]
    return [t.cpu().numpy() for t in (mean, std, om, osd)], torch.cat(pack).cpu().numpy()


def _network():
    def make():
        stats, weights = _once("trained", _train_torch)
        m = learned.Mlp(_ctx(), 24, *stats)
        m.set_params(weights)
        return m
    return _once("mlp", make)


# ---- cases ------------------------------------------------------------------------------------------------

def prepare(case, seed):
    gen = _gen(seed)
    s = dict(case, ctx=_ctx())
    kind, n = case["kind"], case["n"]
    if kind == "invert":
        s["inst"] = _inst(case["inst"])
        s["obs"] = _observe(case["inst"], n, gen)[1]
        s["W"] = _weights(case["inst"], n, case["wpp"], gen)
    elif kind == "batches":  # the fine spectra first, as the entry point advises
        s["batches"] = [dict(inst=_inst(i), stokes=_observe(i, m, gen)[1], W=_weights(i, m, False, gen))
                        for i, m in (("fine", n), ("hmi", case["n2"]))]
    elif kind == "learned":
        s["inst"], s["mlp"] = _inst("hmi"), _network()
        s["obs"], s["W"] = _observe("hmi", n, gen)[1], _weights("hmi", n, False, gen)
    elif kind == "synth":
        s["inst"] = _inst(case["inst"])
        s["models"] = _draw_models(n, gen)
        s["eps"] = (SIGMA * torch.randn((n, 4, _N_OBS[case["inst"]]), generator=gen, device=DEV)
                    if case["noise"] else None)
    elif kind == "train":
        P, S = _observe("hmi", n, gen)
        s["P"], s["X"] = P, S.reshape(n, 24)
        s["ctrl_P"], s["ctrl_X"] = P[:4096].clone(), s["X"][:4096].clone()
        stats = [t.cpu().numpy() for t in (s["X"].mean(0), s["X"].std(0), P[:, 3:].mean(0), P[:, 3:].std(0))]
        s["seed"] = int(seed) % 1000003
        s["mlp"] = learned.Mlp(s["ctx"], 24, *stats, seed=s["seed"])
    elif kind == "classical":
        s["inst"] = _inst("hmi")
        s["obs"] = _observe("hmi", n, gen)[1]
        s["mu"] = torch.rand(n, generator=gen, device=DEV)
    return s


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "invert":
        return vf.invert(ctx, s["inst"], s["obs"], s["W"])
    if kind == "batches":
        return vf.invert_batches(ctx, s["batches"])
    if kind == "learned":
        return learned.invert_learned(ctx, s["inst"], s["mlp"], s["obs"], s["W"])
    if kind == "synth":
        return vf.synthesize(ctx, s["inst"], s["models"], noise=s["eps"], jac=s["jac"])
    if kind == "train":
        r = learned.train_network(ctx, s["mlp"], s["X"], s["P"], s["ctrl_X"], s["ctrl_P"], epochs=1,
                                  batch=s["batch"], lr=1e-3, seed=s["seed"])
        return dict(weights=s["mlp"].get_params(), steps=r["steps"], mse=r["history"][0][1:])
    p, pol = vf.init_classical(ctx, s["inst"], s["obs"])
    return dict(params=p, pol=pol, W=vf.stokes_weights(ctx, s["inst"], s["obs"], s["mu"]))


# Operations a pixel's fit needs (counted per synthesis, Jacobian and step of the method): values of one
# synthesis, derivatives with the normal equations, chi^2 and the damped solve; and the trials and Jacobians
# a fit takes from the default model or from the network's start.
_SYNTH, _JAC, _STEP = ({"hmi": 16356, "fine": 125585}, {"hmi": 79074, "fine": 664568}, {"hmi": 742, "fine": 2514})
_TRIALS, _JACS = {"hmi": 41.5, "fine": 37.7, "learned": 12.8}, {"hmi": 14.5, "fine": 13.5, "learned": 6.8}
_NET_FLOPS = 2 * (24 * 256 + 2 * 256 * 256 + 256 * 10)


def _fit_work(inst, n, wpp, how=None):
    how = how or inst
    flops = (_TRIALS[how] + 1) * (_SYNTH[inst] + _STEP[inst]) + _JACS[how] * _JAC[inst]
    return n * (16 * _N_OBS[inst] * (2 if wpp else 1) + 56), n * flops


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "invert":
        b, f = _fit_work(case["inst"], n, case["wpp"])
    elif kind == "batches":
        (b, f), (b2, f2) = _fit_work("fine", n, False), _fit_work("hmi", case["n2"], False)
        b, f = b + b2, f + f2
    elif kind == "learned":
        b, f = _fit_work("hmi", n, False, "learned")
        f += n * _NET_FLOPS
    elif kind == "synth":
        rows = 4 * _N_OBS[case["inst"]]
        b = n * (40 + 4 * rows * (1 + (10 if case["jac"] else 0) + (1 if case["noise"] else 0)))
        f = n * (_SYNTH[case["inst"]] + (_JAC[case["inst"]] if case["jac"] else 0))
    elif kind == "train":
        rows = n // case["batch"] * case["batch"]
        b, f = rows * (24 + 10) * 4, rows * 3 * _NET_FLOPS
    else:
        b, f = n * (96 + 40 + 4 + 4 + 96), n * 600
    return dict(bytes=float(b), flops=float(f))


def exact(case, seed):
    if case["kind"] == "synth":
        s, spec = prepare(case, seed), _SPECS[case["inst"]]()
        P, n = s["models"].double(), case["n"]
        step = 16384 if case["inst"] == "hmi" else 4096
        S = _chunks(lambda i, j: _forward(spec, P[i:j]), n, step)
        if s["eps"] is not None:
            S = S + s["eps"].double()
        if not case["jac"]:
            return S
        cols = []
        for q, h in enumerate((0.1, 1e-2, 1e-2, 1e-4, 1e-3, 1e-5, 1e-3, 1e-4, 1e-4, 1e-4)):
            d = torch.zeros(10, device=DEV, dtype=torch.float64)
            d[q] = h
            # five-point differences of the 64-bit synthesis
            cols.append(_chunks(lambda i, j: (8.0 * (_forward(spec, P[i:j] + d) - _forward(spec, P[i:j] - d))
                                              - _forward(spec, P[i:j] + 2 * d) + _forward(spec, P[i:j] - 2 * d))
                                / (12.0 * h), n, step))
        return S, torch.stack(cols, -1)
    if case["kind"] == "classical":
        s = prepare(case, seed)
        return _classical64(s["obs"].double(), s["mu"].double())
    return None


def _classical64(S, mu):
    lam0, geff, fine, filt = _hmi_spec()
    x = torch.as_tensor((filt * fine).sum(1) / filt.sum(1), device=DEV)
    cz, lam = 4.66685e-10 * geff * lam0 * lam0, lam0 * 1000.0
    I, Q, U, V = S.unbind(1)
    Ic = I.max(1).values
    d = Ic[:, None] - I
    lo, hi = torch.tensor((0, 0, 1, 2, 3, 4), device=DEV), torch.tensor((1, 2, 3, 4, 5, 5), device=DEV)
    I1 = (I[:, hi] - I[:, lo]) / (x[hi] - x[lo])
    c = torch.tensor((1, 1, 2, 3, 4, 4), device=DEV)
    h0, h1 = x[c] - x[c - 1], x[c + 1] - x[c]
    I2 = 2.0 * (h0 * I[:, c + 1] - (h0 + h1) * I[:, c] + h1 * I[:, c - 1]) / (h0 * h1 * (h0 + h1))
    bl = -(V * I1).sum(1) / (cz * (I1 * I1).sum(1)) / 0.6
    L = torch.sqrt(Q * Q + U * U)
    bt = torch.sqrt(4.0 * (L * I2.abs()).sum(1) / (cz * cz * (I2 * I2).sum(1)) / 0.6)
    P = torch.tensor(DEFAULT_MODEL, device=DEV, dtype=torch.float64).repeat(len(S), 1)
    P[:, 0] = torch.sqrt(bl * bl + bt * bt).clamp(0.0, 5000.0)
    P[:, 1] = torch.rad2deg(torch.atan2(bt, bl))
    P[:, 2] = torch.rad2deg(0.5 * torch.atan2(U.sum(1), Q.sum(1))).remainder(180.0)
    P[:, 3] = (299792.458 * (d * x).sum(1) / d.sum(1) / lam).clamp(-20.0, 20.0)
    P[:, 7], P[:, 8] = 0.3 * Ic, 0.7 * Ic
    pol = torch.sqrt(L * L + V * V).max(1).values / Ic
    icm = torch.full_like(mu, 0.59943)
    for k in (-1.89979, 2.45050, -1.79238, 1.30590, 0.33644):
        icm = icm * mu + k
    W = torch.full_like(S, 1e6)
    W[:, 0] = ((0.7778 * (icm - Ic).abs() + 0.3) ** 2 * 1e6)[:, None]
    return dict(params=P, pol=pol, W=W)
