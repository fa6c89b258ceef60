"""The work this library is used for, as cases that can be timed and compared.

Each case is one call (or one short run of calls) through the public binding,
with synthetic lenses and proposals of the shapes that the library's workload
generators draw: a 64x64 px image without supersampling up to 200x200 px at
4x4 sub-pixels, Gaussian and Moffat PSFs of 11 to 41 px, one proposal up to
tens of thousands, every convolution precision, both mass models, explicit
and solved amplitudes, and the calls that carry them (host and device
buffers, many lenses, serving, the device-resident sampler).

The model images and likelihoods of exact() are a plain FP64 evaluation in
torch of the same equations (Cao et al. 2025, Sec. 2.1-2.4), which also makes
the mock observations.
"""
import math

import numpy as np
import torch

from paper_2503_08586_amd import binding, synth

PREC = {"fp32": binding.LENS_PREC_FP32, "f16": binding.LENS_PREC_F16_SPLIT, "bf16": binding.LENS_PREC_BF16,
        "split3": binding.LENS_PREC_BF16_SPLIT3}
LIGHT = {"both": 0, "lens": 1, "source": 2, "double": 3}
CHANNELS = {"both": 2, "lens": 1, "source": 1, "double": 4}
MASK_RADIUS = 3.0   # arcsec


def _case(name, call, **kw):
    c = {"name": name, "call": call, "lenses": 1, "n": 1, "px": 128, "dpix": 0.05, "s": 4, "k": 21, "psf": "gaussian",
         "fwhm": 0.10, "prec": "fp32", "mass": "sie", "light": "explicit", "stage": "prior", "mixed": False}
    c.update(kw)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # a single model of a small cut-out (no supersampling), as an optimiser or a notebook asks for it
        _case("one_64px", "host", n=1, px=64, dpix=0.074, s=1, k=11, fwhm=0.15),
        # a host sampler's batch of live points on a survey-scale lens (the odd size such a batch has)
        _case("live_points_128px", "host", n=301, stage="posterior"),
        # a full device batch on a survey-scale lens: the throughput of one fit
        _case("full_128px", "device", n=65536),
        # a small device batch on a large image with a wide PSF, matrix-core convolution
        _case("batch64_200px_f16", "device", n=64, px=200, k=41, psf="moffat", fwhm=0.15, prec="f16"),
        # many large lenses in one launch, FP16 matrix-core convolution: a survey's throughput
        _case("multi16_200px_f16", "multi_device", lenses=16, n=1000, px=200, k=41, psf="moffat", fwhm=0.15, prec="f16"),
        # uneven lenses (48-160 px, s of 2 or 4, PSF 11-31) from host buffers, FP32 convolution
        _case("mix24_host", "multi", lenses=24, n=700, mixed=True),
        # amplitudes solved per proposal, one component per galaxy, the amplitudes returned
        _case("amps_128px", "amps", n=777, light="both", stage="posterior"),
        # two components per galaxy, solved amplitudes
        _case("double_128px", "device", n=2500, light="double"),
        # the elliptical power law instead of the isothermal ellipsoid
        _case("power_law_128px", "device", n=4096, mass="epl"),
        # a 64-walker ensemble advanced on the device, its chain returned
        _case("sampler64_128px", "sampler", n=64, iters=4, stage="posterior"),
        # one small ensemble per lens, many lenses together, FP32 convolution
        _case("samplers12_mix", "samplers", lenses=12, n=48, iters=2, mixed=True, stage="posterior"),
        # a burst of requests of mixed size on resident lenses of mixed shape
        _case("serving_mix_f16", "serving", lenses=12, n=1000, requests=24, mixed=True, prec="f16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["host", "device", "device", "multi_device", "multi", "amps", "sampler", "samplers", "serving"])
    c = _case(None, call)
    many = call in ("multi", "multi_device", "samplers", "serving")
    c["lenses"] = rng.randint(3, 24) if many else 1
    c["mixed"] = many and rng.random() < 0.7
    c["px"] = rng.randint(48, 200)
    c["dpix"] = round(rng.uniform(0.05, 0.074), 4)
    c["s"] = rng.choice([1, 2, 4, 4, 4])
    c["k"] = rng.randrange(11, 42, 2)
    c["psf"] = rng.choice(["gaussian", "moffat"])
    c["fwhm"] = round(rng.uniform(0.10, 0.15), 4)
    c["stage"] = rng.choice(["prior", "posterior"])
    if call == "amps":
        c["light"] = rng.choice(["both", "both", "double", "lens", "source"])
    elif call in ("device", "multi_device") and rng.random() < 0.3:
        c["light"] = rng.choice(["both", "double", "source"])
    else:
        c["prec"] = rng.choice(["fp32", "fp32", "f16", "f16", "bf16", "split3"])
    if rng.random() < 0.25 and c["light"] != "lens":
        c["mass"] = "epl"
    if call in ("sampler", "samplers"):
        c["n"] = 2 * _log_int(rng, 8, 256 if call == "sampler" else 48)
        c["iters"] = rng.randint(1, 6)
        c["stage"] = "posterior"
        c["light"] = "explicit"
    else:
        c["n"] = _log_int(rng, 1, 16384 if call in ("host", "device", "amps") else 2000)
    if call == "serving":
        c["requests"] = rng.randint(4, 30)
    # no dearer than the largest listed case
    cap = 0.8 * _cost(_case("", "device", n=65536))
    while c["n"] > 2 and _cost(c) > cap:
        c["n"] = max(2, c["n"] // 4 * 2)
    return c


def _evals(case):
    """Proposals evaluated in one pass."""
    if case["call"] == "serving":
        return case["requests"] * case["n"]
    if case["call"] in ("sampler", "samplers"):
        return case["lenses"] * case["n"] * case["iters"]
    return case["lenses"] * case["n"]


def _pixels(px, dpix, k):
    """(masked pixels, pixels in the mask's PSF footprint), nearly."""
    m = min(px * px, math.pi * (MASK_RADIUS / dpix) ** 2)
    return m, min(px * px, math.pi * (MASK_RADIUS / dpix + (k - 1) / 2) ** 2)


def _per_proposal(case):
    px = 104 if case["mixed"] else case["px"]
    masked, needed = _pixels(px, case["dpix"], case["k"])
    # per sub-pixel: ray trace, lens equation and one Sersic profile per light component; the
    # power law adds its angular function; per masked pixel one multiply-add per PSF tap and component
    light = case["light"]
    comps = CHANNELS.get(light, 2)
    sub = (50 if light != "lens" else 0) + 32 * comps + (60 if case["mass"] == "epl" else 0)
    chan = 1 if light == "explicit" else comps
    return needed * case["s"] ** 2 * sub, masked * chan * 2.0 * case["k"] ** 2, masked


def _cost(case):
    a, b, _ = _per_proposal(case)
    return _evals(case) * (a + 0.5 * b) * (1.7 if case["mass"] == "epl" else 1.0)


def work(case):
    a, b, masked = _per_proposal(case)
    n = _evals(case)
    out = 8 * (1 + (CHANNELS.get(case["light"], 2) if case["call"] == "amps" else 0))
    return {"flops": n * (a + b), "bytes": n * (20 * 8 + out) + case["lenses"] * masked * 8}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
LO = np.array([b[1] for b in synth.PRIOR_BOX] + [0.0])
HI = np.array([b[2] for b in synth.PRIOR_BOX] + [0.0])


def _box(case):
    lo, hi = LO.copy(), HI.copy()
    if case["mass"] == "epl":
        lo[19], hi[19] = 1.6, 2.4
    return lo, hi


def _proposals(case, rng, truth, n):
    lo, hi = _box(case)
    if case["stage"] == "prior":
        p = lo + (hi - lo) * rng.random((n, 20))
    else:   # a sampler that has found the posterior
        p = np.clip(truth + 0.004 * (hi - lo) * rng.normal(size=(n, 20)), lo, hi)
    if case["light"] == "double":   # R_e of the second components in the n slots
        p[:, synth.SLOT["n_l"]] = p[:, synth.SLOT["R_l"]] * rng.uniform(0.3, 3.0, n)
        p[:, synth.SLOT["n_s"]] = p[:, synth.SLOT["R_s"]] * rng.uniform(0.3, 3.0, n)
    return np.ascontiguousarray(p)


def _inputs(case, seed):
    """Every lens of the case (geometry, PSF, noise, truth, mock data) and its proposals, from the seed."""
    rng = np.random.default_rng([seed, 2503])
    # the shapes of a mixed set belong to the case, as the lenses of a survey do; the seed draws what is on them
    shapes = np.random.default_rng([case["lenses"], case["px"], case["k"], 86])
    specs = []
    for _ in range(case["lenses"]):
        px, dpix, s, k, fwhm, psf = case["px"], case["dpix"], case["s"], case["k"], case["fwhm"], case["psf"]
        if case["mixed"]:
            px, dpix = int(shapes.integers(48, 161)), float(shapes.uniform(0.05, 0.074))
            s, k = int(shapes.choice([2, 4])), int(shapes.choice(np.arange(11, 32, 2)))
            fwhm = float(shapes.uniform(0.10, 0.15))
        psf = synth.gaussian_psf(k, fwhm, dpix) if psf == "gaussian" else synth.moffat_psf(k, fwhm, 3.0, dpix)
        lo, hi = _box(case)
        truth = lo + (hi - lo) * (0.1 + 0.8 * rng.random(20))
        if case["light"] == "double":
            truth[synth.SLOT["n_l"]] = truth[synth.SLOT["R_l"]] * rng.uniform(0.5, 2.0)
            truth[synth.SLOT["n_s"]] = truth[synth.SLOT["R_s"]] * rng.uniform(0.5, 2.0)
        sigma = np.full((px, px), 0.01)
        noise = rng.normal(0.0, 1.0, (px, px)) * sigma
        n = case["n"]
        if case["mixed"] and case["call"] == "multi":
            n = max(1, int(shapes.integers(max(1, n // 8), 2 * n)))
        spec = synth.LensSpec(px, px, dpix, s, psf, sigma, synth.circular_mask(px, px, dpix, MASK_RADIUS), truth,
                              _proposals(case, rng, truth, n), noise)
        spec.data = _truth_image(case, spec) + noise
        specs.append(spec)
    reqs = []
    for _ in range(case.get("requests", 0)):
        j = int(shapes.integers(0, len(specs)))
        n = max(1, int(shapes.integers(max(1, case["n"] // 10), 2 * case["n"])))
        reqs.append((j, _proposals(case, rng, specs[j].truth, n)))
    return specs, reqs


class _State:
    """The handles a program keeps: one context for the process, its lenses and ensembles."""
    ctx = None

    def __init__(self, case):
        if _State.ctx is None:
            _State.ctx = binding.LensContext(0)
        self.case, self.lids, self.ens = case, [], []

    def __del__(self):
        for e in self.ens:
            _State.ctx.ensemble_destroy(e)
        for lid in self.lids:
            _State.ctx.unload(lid)


def prepare(case, seed):
    specs, reqs = _inputs(case, seed)
    st = _State(case)
    ctx, light = st.ctx, case["light"]
    for sp in specs:
        st.lids.append(ctx.load(sp, precision=PREC[case["prec"]], amplitudes=int(light != "explicit"),
                                light_model=LIGHT.get(light, 0), sersic_n=synth.DOUBLE_SERSIC_N,
                                mass_model=int(case["mass"] == "epl")))
    st.props = [sp.proposals for sp in specs]
    st.counts = [p.shape[0] for p in st.props]
    st.reqs = reqs
    if case["call"] in ("device", "multi_device"):
        st.dev = torch.from_numpy(np.concatenate(st.props)).cuda()
        st.out = torch.zeros(st.dev.shape[0], dtype=torch.float64, device="cuda")
    if case["call"] in ("sampler", "samplers"):
        lo, hi = _box(case)
        for lid, p in zip(st.lids, st.props):
            st.ens.append(ctx.ensemble(lid, p, lo, hi, stretch=2.0, seed=seed))
    return st


def run(st):
    ctx, call = st.ctx, st.case["call"]
    if call == "host":
        return ctx.loglike(st.lids[0], st.props[0])
    if call == "amps":
        return ctx.loglike_amps(st.lids[0], st.props[0])
    if call == "device":
        ctx.loglike_device(st.lids[0], st.dev, st.out)
        return st.out
    if call == "multi_device":
        ctx.loglike_multi_device(st.lids, st.counts, st.dev, st.out)
        return st.out
    if call == "multi":
        return ctx.loglike_multi(st.lids, st.props)
    if call == "sampler":
        return ctx.ensemble_run(st.ens[0], st.case["iters"], thin=1, chain=True)
    if call == "samplers":
        return ctx.ensemble_run_many(st.ens, st.case["iters"], thin=1, chain=True)
    reqs = [ctx.submit(st.lids[j], p) for j, p in st.reqs]
    for r in reqs:
        ctx.wait(r)
    return [r.out for r in reqs]


# ---------------------------------------------------------------------------
# the same likelihood in plain FP64
# ---------------------------------------------------------------------------
def _sersic_b(n):
    """b with P(2n, b) = 1/2 (Eq. 9), by bisection."""
    lo, hi = torch.zeros_like(n), 2.0 * n + 1.0
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        below = torch.special.gammainc(2.0 * n, mid) < 0.5
        lo, hi = torch.where(below, mid, lo), torch.where(below, hi, mid)
    return 0.5 * (lo + hi)


def _col(p, i):
    return p[:, i].reshape(-1, 1, 1)


def _radius(dx, dy, q, phi):
    """R_p of Eq. 10."""
    c, s = torch.cos(phi), torch.sin(phi)
    u, v = c * dx + s * dy, c * dy - s * dx
    return torch.sqrt(q * u * u + v * v / q)


def _profile(r, re, n, b):
    return torch.exp(-b * ((r / re) ** (1.0 / n) - 1.0))


def _channels(case, spec, p):
    """PSF-convolved images [n, components, ny, nx] of proposals p at unit amplitude."""
    dev, f8 = p.device, torch.float64
    ny, nx, s = spec.ny, spec.nx, spec.s
    gy = ((torch.arange(ny * s, dtype=f8, device=dev) - 0.5 * (ny * s - 1)) * (spec.dpix / s)).reshape(1, -1, 1)
    gx = ((torch.arange(nx * s, dtype=f8, device=dev) - 0.5 * (nx * s - 1)) * (spec.dpix / s)).reshape(1, 1, -1)
    light = case["light"]
    tE, q, phi = _col(p, 0), _col(p, 1), _col(p, 2)
    dx, dy = gx - _col(p, 3), gy - _col(p, 4)
    double = light == "double"
    fixed = [torch.full_like(tE, v) for v in synth.DOUBLE_SERSIC_N]
    images = []
    if light != "source":
        r = _radius(dx, dy, _col(p, 10), _col(p, 11))
        for j, re in enumerate((_col(p, 8), _col(p, 9)) if double else (_col(p, 8),)):
            n = fixed[j] if double else _col(p, 9)
            images.append(_profile(r, re, n, _sersic_b(n)))
    if light != "lens":
        c, sn = torch.cos(phi), torch.sin(phi)
        x1, x2 = c * dx + sn * dy, c * dy - sn * dx
        psi = torch.sqrt(q * q * x1 * x1 + x2 * x2)
        if case["mass"] == "sie":
            e = torch.sqrt(1.0 - q * q)
            a1 = tE * torch.sqrt(q) / e * torch.atan(e * x1 / psi)
            a2 = tE * torch.sqrt(q) / e * torch.atanh(e * x2 / psi)
        else:   # Tessore & Metcalf (2015): the angular function as its series
            t = _col(p, 19) - 1.0
            f = (1.0 - q) / (1.0 + q)
            z = torch.complex(q * x1 / psi, x2 / psi)
            w, term, tot = z * z, z, z
            for j in range(1, 2 + int(math.log(1e-18) / math.log(max(1e-3, float(f.max()))))):
                term = term * (w * (-f * (2.0 * j - 2.0 + t) / (2.0 * j + 2.0 - t)))
                tot = tot + term
            tot = tot * (2.0 / (1.0 + q) * (tE * torch.sqrt(q)) ** t * psi ** (1.0 - t))
            a1, a2 = tot.real, tot.imag
        g1, g2 = _col(p, 5), _col(p, 6)
        bx = gx - (c * a1 - sn * a2) + (g1 * gx + g2 * gy)
        by = gy - (sn * a1 + c * a2) + (g2 * gx - g1 * gy)
        r = _radius(bx - _col(p, 17), by - _col(p, 18), _col(p, 15), _col(p, 16))
        for j, re in enumerate((_col(p, 13), _col(p, 14)) if double else (_col(p, 13),)):
            n = fixed[2 + j] if double else _col(p, 14)
            images.append(_profile(r, re, n, _sersic_b(n)))
    img = torch.stack(images, 1)
    img = img.reshape(img.shape[0], img.shape[1], ny, s, nx, s).mean(dim=(3, 5))
    # PSF: out[y, x] = sum K[a, b] img[y - a + r, x - b + r], one PSF row at a time as a product
    # with the banded matrix of that row
    k, r = spec.k, (spec.k - 1) // 2
    psf = torch.from_numpy(spec.psf).to(dev)
    at = torch.arange(nx, device=dev).reshape(1, -1) - torch.arange(nx, device=dev).reshape(-1, 1) + r
    inside, at = (at >= 0) & (at < k), at.clamp(0, k - 1)
    out = torch.zeros_like(img)
    for a in range(k):
        band = torch.where(inside, psf[a][at], torch.zeros_like(psf[0, 0]))
        d = a - r
        y0, y1 = max(0, d), min(ny, ny + d)
        if y0 < y1:
            out[:, :, y0:y1] += img[:, :, y0 - d:y1 - d] @ band
    return out


def _amplitudes(case, p):
    return torch.stack([p[:, 7], p[:, 12]], 1)


def _truth_image(case, spec):
    p = torch.from_numpy(spec.truth[None]).cuda()
    ch = _channels(case, spec, p)[0]
    a = {"lens": [spec.truth[7]], "source": [spec.truth[12]],
         "double": [spec.truth[7], 0.6 * spec.truth[7], spec.truth[12], 0.6 * spec.truth[12]]}
    a = torch.tensor(a.get(case["light"], [spec.truth[7], spec.truth[12]]), dtype=torch.float64, device=ch.device)
    return (a.reshape(-1, 1, 1) * ch).sum(0).cpu().numpy()


def _nnls(F, g):
    """Amplitudes >= 0 that minimise s.F s - 2 s.g, over every support."""
    n, m = g.shape
    best, best_s = torch.zeros(n, dtype=g.dtype, device=g.device), torch.zeros_like(g)
    for S in range(1, 1 << m):
        idx = [i for i in range(m) if S >> i & 1]
        sub = F[:, idx][:, :, idx]
        s, info = torch.linalg.solve_ex(sub, g[:, idx].unsqueeze(-1))
        s = s.squeeze(-1)
        gain = (s * g[:, idx]).sum(1)
        ok = (info == 0) & (s >= 0).all(1) & (gain > best)
        full = torch.zeros_like(g)
        full[:, idx] = s
        best = torch.where(ok, gain, best)
        best_s = torch.where(ok.unsqueeze(1), full, best_s)
    return best_s


def _loglike(case, spec, props):
    """(lnL [n], amplitudes [n, components])."""
    dev = torch.device("cuda")
    p = torch.from_numpy(props).to(dev)
    use = torch.from_numpy(spec.mask.astype(bool)).to(dev)
    d = torch.from_numpy(spec.data).to(dev)[use]
    sg = torch.from_numpy(spec.sigma).to(dev)[use]
    norm = -0.5 * torch.log(2.0 * math.pi * sg * sg).sum()
    sub = spec.ny * spec.nx * spec.s ** 2 * (2 if case["mass"] == "epl" else 1)
    step = max(1, int(4e7 / sub))
    ls, amps = [], []
    for i in range(0, p.shape[0], step):
        q = p[i:i + step]
        ch = _channels(case, spec, q)[..., use]
        if case["light"] == "explicit":
            a = _amplitudes(case, q)
        else:
            w = ch / sg
            F = torch.stack([(w * w[:, j:j + 1]).sum(-1) for j in range(w.shape[1])], 1)
            a = _nnls(F, (w * (d / sg)).sum(-1))
        res = (d - (a.unsqueeze(-1) * ch).sum(1)) / sg
        ls.append(norm - 0.5 * (res * res).sum(-1))
        amps.append(a)
    return torch.cat(ls), torch.cat(amps)


def exact(case, seed):
    call = case["call"]
    if call in ("sampler", "samplers"):   # a chain of random moves: its proposals are the sampler's own
        return None
    specs, reqs = _inputs(case, seed)
    if call == "serving":
        return [_loglike(case, specs[j], p)[0].cpu().numpy() for j, p in reqs]
    got = [_loglike(case, sp, sp.proposals) for sp in specs]
    if call == "host":
        return got[0][0].cpu().numpy()
    if call == "amps":
        return got[0][0].cpu().numpy(), got[0][1].cpu().numpy()
    if call == "multi":
        return [g[0].cpu().numpy() for g in got]
    return torch.cat([g[0] for g in got])
