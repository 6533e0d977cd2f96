"""The calls whose speed is followed: what a user of the library has it do, over the range of sizes.

listed() names the calls, draw() gives more of the same ranges, prepare() makes a call's inputs and
the context that a program keeps, run() is one pass through the public entry points, work() the bytes
and operations it cannot do without, and exact() its results in 64 bits from plain torch.

The inputs follow the library's own synthetic recipe: 12 x 94 SSP spectra, Gaussian bands of 400 A
between 3600 and 9700 A, galaxies drawn uniformly per parameter.  Observations are the magnitudes of
a true galaxy plus noise of 0.03 to 0.2 mag, and the parameters of a call lie around that truth, as a
sampler's or an optimiser's do.
"""
import functools
import math

import numpy as np
import torch

import paper_2506_19919_amd as sps

N_MET, N_AGE, N_SSP = 12, 94, 12 * 94
N_Z, Z_LO, Z_HI = 64, 0.1, 3.0
SIGMA_A, SIGMA_LOGZ, BURST_DLOGT = 400.0, 0.2, 0.3
H0, OM = 70.0, 0.3
PREC = {"f64": sps.SPS_F64, "f32": sps.SPS_F32, "bf16x": sps.SPS_BF16X}
SFH = {"dpl": sps.SPS_SFH_DPL, "lognormal": sps.SPS_SFH_LOGNORMAL}
# bounds of the unbounded samplers' parameters, and the ranges that galaxies are drawn from
BOUNDS = [[8.0, 12.5], [0.1, 14.0], [0.1, 8.0], [0.1, 8.0], [0.0, 0.2], [4.5, 8.5], [-2.0, 0.4], [0.0, 4.0],
          [-1.5, 0.0], [0.0, 0.5]]
DRAWN = {"dpl": [[9.0, 11.5], [1.0, 12.0], [0.5, 5.0], [0.5, 5.0], [0.0, 0.1], [5.0, 8.0], [-1.5, 0.2], [0.0, 2.0],
                 [-1.0, -0.4], [0.0, 0.3]],
         "lognormal": [[9.0, 11.5], [1.0, 12.0], [0.2, 1.5], [0.0, 0.0], [0.0, 0.1], [5.0, 8.0], [-1.5, 0.2],
                       [0.0, 2.0], [-0.7, -0.7], [0.0, 0.0]]}
TRUTHS = 2048   # distinct true galaxies of a batch; larger batches repeat them at other masses


def listed():
    return [
        # one galaxy: the step of an optimiser or of a sampler outside the library
        dict(name="loglike_1", op="loglike", n=1, n_band=6, sfh="dpl"),
        # a few hundred walkers of an outside sampler on the unbounded parameters, ragged
        dict(name="logpost_250", op="logpost", n=250, n_band=6, sfh="dpl"),
        # one served batch of galaxies
        dict(name="loglike_4096", op="loglike", n=4096, n_band=6, sfh="dpl"),
        # training through the magnitudes (forward and backward), all 8 bands, ragged
        dict(name="vjp_30011", op="vjp", n=30011, n_band=8, sfh="dpl"),
        # a forward catalogue of log-normal galaxies with bursts
        dict(name="mags_100k", op="mags", n=100_000, n_band=6, sfh="lognormal"),
        # the likelihood sweep of a survey
        dict(name="loglike_1m", op="loglike", n=1_000_000, n_band=6, sfh="dpl"),
        # the double-precision reference photometry
        dict(name="exact_f64_64", op="exact_mags", n=64, n_band=6, sfh="lognormal", prec="f64", n_wave=2000),
        # spectrum-level likelihood with its gradient, in both precisions
        dict(name="exact_bf16x_4096", op="exact_loglike", n=4096, n_band=6, sfh="dpl", prec="bf16x", n_wave=5000),
        dict(name="exact_f32_4096", op="exact_loglike", n=4096, n_band=6, sfh="dpl", prec="f32", n_wave=5000),
        # training through spectrum-level magnitudes, a ragged batch
        dict(name="exact_vjp_20011", op="exact_vjp", n=20011, n_band=6, sfh="dpl", prec="bf16x", n_wave=2000),
        # a block of sampler iterations: a small target list, and a full card
        dict(name="hmc_128x4", op="hmc", n=128, n_band=6, sfh="dpl", n_chain=4, n_leapfrog=10, n_warmup=3, n_sample=5),
        dict(name="hmc_16384x4", op="hmc", n=16384, n_band=6, sfh="dpl", n_chain=4, n_leapfrog=10, n_warmup=2,
             n_sample=4),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["loglike", "loglike", "logpost", "vjp", "mags", "exact_mags", "exact_loglike", "exact_vjp", "hmc"])
    c = dict(op=op, n_band=rng.randint(1, 8), sfh=rng.choice(["dpl", "dpl", "lognormal"]))
    if op == "loglike":
        c["n"] = size(1, 1_000_000)
    elif op in ("logpost", "vjp", "mags"):
        c["n"] = size(1, 100_000)
    elif op == "exact_mags" and rng.random() < 0.4:
        c.update(n=size(1, 500), prec="f64", n_wave=rng.randint(500, 2500))
    elif op.startswith("exact"):
        c.update(n=size(16, 4096), prec=rng.choice(["f32", "bf16x"]), n_wave=rng.randint(500, 5000))
    else:
        c.update(n=size(16, 1024), sfh="dpl", n_band=6, n_chain=rng.randint(2, 6), n_leapfrog=rng.randint(3, 12),
                 n_warmup=rng.randint(0, 3), n_sample=rng.randint(2, 5))
    return c


# ------------------------------------------------------------------ tables
@functools.lru_cache(maxsize=2)
def ssp_grid(n_wave):
    """Synthetic SSP spectra [met][age][wave] in Lsun / A per Msun: two Planck curves with 5 % noise."""
    met = -2.0 + 2.4 * np.arange(N_MET) / (N_MET - 1)
    age = 5.5 + 0.05 * np.arange(N_AGE)
    wave = 10.0 ** (2.0 + 3.0 * np.arange(n_wave) / (n_wave - 1))
    z, a, lam = met[:, None, None], age[None, :, None], wave[None, None, :]

    def planck(t):
        x = 1.438777e8 / (lam * t)
        with np.errstate(over="ignore"):
            return (15.0 / np.pi ** 4) * x ** 4 / (lam * np.expm1(x))

    hot = 1.0 / (1.0 + 10.0 ** (a - 8.0))
    lum = 10.0 ** (3.0 - 0.8 * (a - 5.5)) * (hot * planck(10.0 ** (4.6 - 0.22 * (a - 5.5)) * (1.0 + 0.05 * z))
                                             + (1.0 - hot) * planck(10.0 ** (3.75 - 0.05 * (a - 5.5)) * (1.0 + 0.05 * z)))
    lum = lum * np.exp(0.05 * np.random.default_rng(1).standard_normal(lum.shape))
    return dict(log10_met=met, log10_age_yr=age, wave_A=wave, lum=np.ascontiguousarray(lum))


def filters(n_band):
    b = np.arange(n_band)
    centre = 3600.0 * (9700.0 / 3600.0) ** (b / max(n_band - 1, 1))
    return dict(center_A=centre, sigma_A=np.full(n_band, SIGMA_A))


@functools.lru_cache(maxsize=1)
def context(n_wave, n_band, prec, rows, exact_rows):
    """The handle a program keeps: tables on the card, the z table, workspaces for its largest call."""
    ctx = sps.Context(ssp_grid(n_wave), filters(n_band), precisions=(sps.SPS_F64, PREC[prec]), max_gal=rows,
                      max_exact=exact_rows)
    ctx.build_ztable(N_Z, Z_LO, Z_HI)
    return ctx


def n_wave_of(case):
    return case.get("n_wave", 2000)


def the_context(case):
    rows = case["n"] * case.get("n_chain", 1)
    return context(n_wave_of(case), case["n_band"], case.get("prec", "f64"), rows, rows if "prec" in case else 0)


# ------------------------------------------------------------------ the model in 64 bits, plain torch
def dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def f64(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=dev())


@functools.lru_cache(maxsize=2)
def model(n_wave, n_band, table):
    """Constants of the forward model; table: with the z table (approximate photometry)."""
    g, f = ssp_grid(n_wave), filters(n_band)
    la, lz, lam = g["log10_age_yr"], g["log10_met"], g["wave_A"]
    mid = 0.5 * (la[1:] + la[:-1])
    trap = 0.5 * (np.append(lam[1:], lam[-1]) - np.insert(lam[:-1], 0, lam[0]))
    m = dict(edges=f64(np.concatenate([[0.0], 10.0 ** (mid - 9.0), [np.inf]])),
             ledges=f64(np.concatenate([[-np.inf], mid, [np.inf]])), zedges=f64(0.5 * (lz[1:] + lz[:-1])),
             wave=f64(lam), trap=f64(trap), centre=f64(f["center_A"]), lum=f64(g["lum"].reshape(N_SSP, n_wave)))
    if table:
        z = Z_LO + (Z_HI - Z_LO) / (N_Z - 1) * torch.arange(N_Z, dtype=torch.float64, device=dev())
        t = torch.exp(-0.5 * (((1 + z)[:, None, None] * m["wave"] - m["centre"][:, None]) / SIGMA_A) ** 2)
        norm = (t * (m["trap"] / m["wave"])).sum(-1, keepdim=True)
        m["table"] = (t * (m["wave"] * m["trap"]) / norm) @ m["lum"].T     # [n_z][n_band][n_ssp]
    return m


def gauss(n):
    x, w = np.polynomial.legendre.leggauss(n)
    return f64(x), f64(w)


def cosmology(z):
    """Age of the universe at z [Gyr] and the distance part of the AB magnitude (flat LCDM)."""
    mpc_km, gyr_s, c_kms = 3.0856775814913673e19, 3.15576e16, 299792.458
    ol = 1.0 - OM
    t = 2.0 / (3.0 * H0 / mpc_km * gyr_s * math.sqrt(ol)) * torch.asinh(math.sqrt(ol / OM) * (1 + z) ** -1.5)
    x, w = gauss(32)
    zz = 0.5 * z[:, None] * (1 + x)
    dl = (1 + z) * (c_kms / H0 * 1e-19 * mpc_km * 1e24) * 0.5 * z * (w / torch.sqrt(OM * (1 + zz) ** 3 + ol)).sum(-1)
    k = (1 + z) * 3.828e33 / (4 * math.pi * 2.99792458e18 * 3631.0e-23)
    return t, -2.5 * torch.log10(k) + 5.0 * torch.log10(dl)


def dpl_masses(m, th, t):
    """Mass per age bin of the double power law: Gauss-Legendre panels in X = ln(t / tau)."""
    tau, al, be = (th[p][:, None] for p in (1, 2, 3))
    lo, hi, t = m["edges"][:-1], m["edges"][1:], t[:, None]

    def integral(x_hi, span, tau, al, be, panels, nodes):
        x, w = gauss(nodes)
        c = (torch.arange(panels, dtype=torch.float64, device=x.device)[:, None] + 0.5 * (1 + x)).reshape(-1) / panels
        X = (x_hi - span)[..., None] + span[..., None] * c
        h = tau[..., None] / (torch.exp((al[..., None] - 1) * X) + torch.exp(-(be[..., None] + 1) * X))
        return (h * w.repeat(panels)).sum(-1) * span * (0.5 / panels)

    age = torch.where(lo < t, lo, torch.zeros_like(lo))
    x_hi = torch.log(t - age) - torch.log(tau)
    closed = hi < t
    span = -torch.log1p(-(torch.where(closed, hi, lo) - lo) / (t - age))
    narrow = integral(x_hi, torch.where(closed, span, torch.zeros_like(span)), tau, al, be, 1, 6)
    # the six bins next to t = 0, the open one among them, by many panels
    last = (lo < t).sum(-1, keepdim=True) - 1
    six = (last - torch.arange(6, device=last.device)).clamp(min=0)
    x6, s6, open6 = x_hi.gather(1, six), span.gather(1, six), ~closed.gather(1, six)
    reach = x6 - (torch.minimum(x6, torch.zeros_like(x6)) - 45.0 / (be + 1))
    s6 = torch.where(open6, reach, torch.minimum(s6, reach))
    wide = integral(x6, s6, tau.expand_as(x6), al.expand_as(x6), be.expand_as(x6), 48, 10)
    return torch.where(lo < t, narrow, torch.zeros_like(narrow)).scatter(1, six, wide)


def lognormal_masses(m, th, t):
    """The same for the log-normal SFH, up to a common factor: normal-CDF differences."""
    tp, w = th[1][:, None], th[2][:, None]
    lo, hi, t = m["edges"][:-1], m["edges"][1:], t[:, None]

    def x_at(age):
        left = torch.where(age < t, t - age, torch.ones_like(t))
        return torch.log(left / tp) / w - w

    def tail(x):   # Phi(-x)
        return 0.5 * torch.special.erfc(x / math.sqrt(2.0))

    x_hi, x_lo = x_at(lo), x_at(hi)
    both = torch.where(x_lo > 0, tail(x_lo) - tail(x_hi), tail(-x_hi) - tail(-x_lo))
    mass = torch.where(hi < t, both, tail(-x_hi))
    return torch.where(lo < t, mass, torch.zeros_like(mass))


def weights(m, sfh, th, t):
    """P_age [n][94] and P_Z [n][12]."""
    mass = (dpl_masses if sfh == "dpl" else lognormal_masses)(m, th, t)
    le = torch.minimum(m["ledges"], (torch.log10(t) + 9.0)[:, None])
    u = ((le - th[5][:, None]) / BURST_DLOGT).clamp(-1.0, 1.0)
    u2 = u * u
    cdf = 0.5 + 1.09375 * u * (1 - u2 + u2 * u2 * (0.6 - u2 / 7.0))
    burst = cdf[:, 1:] - cdf[:, :-1]
    fb = th[4][:, None]
    pa = (1 - fb) * mass / mass.sum(-1, keepdim=True) + fb * burst / burst.sum(-1, keepdim=True)
    c = torch.special.ndtr((m["zedges"] - th[6][:, None]) / SIGMA_LOGZ)
    end = torch.ones_like(c[:, :1])
    return pa, torch.cat([c, end], 1) - torch.cat([0 * end, c], 1)


def attenuation(lam, th):
    """F_att at rest-frame wavelengths lam [n][k]."""
    tv, de, fl = (th[p][:, None] for p in (7, 8, 9))
    return fl + (1 - fl) * torch.exp(-tv * (lam / 5500.0) ** de)


def magnitudes(m, sfh, th, z, table):
    t, m0 = cosmology(z)
    pa, pz = weights(m, sfh, th, t)
    if table:
        u = (z - Z_LO) / ((Z_HI - Z_LO) / (N_Z - 1))
        k = u.floor().clamp(0, N_Z - 2).long()
        f = (u - k)[:, None]
        w = (pz[:, :, None] * pa[:, None, :]).reshape(len(z), N_SSP)
        flux = z.new_zeros(len(z), len(m["centre"]))
        for node in torch.unique(torch.cat([k, k + 1])).tolist():
            part = (w @ m["table"][node].T.contiguous())
            share = torch.where((k == node)[:, None], 1 - f, torch.where((k + 1 == node)[:, None], f, torch.zeros_like(f)))
            flux = flux + share * part
        flux = flux * attenuation(m["centre"] / (1 + z)[:, None], th)
    else:
        w = (pz[:, :, None] * pa[:, None, :]).reshape(len(z), N_SSP)
        sed = (w @ m["lum"]) * attenuation(m["wave"][None, :], th) * (m["wave"] * m["trap"])
        flux = []
        for c in m["centre"]:
            tr = torch.exp(-0.5 * (((1 + z)[:, None] * m["wave"] - c) / SIGMA_A) ** 2)
            flux.append((sed * tr).sum(-1) / (tr * (m["trap"] / m["wave"])).sum(-1))
        flux = torch.stack(flux, 1)
    return m0[:, None] - 2.5 * th[0][:, None] - 2.5 * torch.log10(flux)


# ------------------------------------------------------------------ inputs
def prepare(case, seed):
    n, nb, sfh, op = case["n"], case["n_band"], case["sfh"], case["op"]
    ctx = the_context(case)
    d = dev()
    g = torch.Generator(device=d).manual_seed(seed)

    def uniform(*shape):
        return torch.rand(*shape, generator=g, device=d, dtype=torch.float64)

    def normal(*shape):
        return torch.randn(*shape, generator=g, device=d, dtype=torch.float64)

    # true galaxies, their magnitudes, and a batch of them at other masses
    k = min(n, TRUTHS)
    lo, hi = f64(DRAWN[sfh])[:, :1], f64(DRAWN[sfh])[:, 1:]
    truth = lo + (hi - lo) * uniform(10, k)
    z = (Z_LO + (Z_HI - Z_LO) * uniform(k)).float().double().clamp(0.1001, 2.9999)
    m = model(2000, nb, True)
    mags = torch.cat([magnitudes(m, sfh, truth[:, i:i + 256], z[i:i + 256], True) for i in range(0, k, 256)])
    at = torch.arange(n, device=d) % k
    shift = 0.5 * (uniform(n) - 0.5)
    truth, z, mags = truth[:, at], z[at], mags[at] - 2.5 * shift[:, None]
    truth[0] += shift
    sigma = 0.03 + 0.17 * uniform(n, nb)
    obs = (mags + sigma * normal(n, nb)).float()
    rank = uniform(n, nb).argsort(1)
    seen = rank < (min(nb, 3) + (uniform(n, 1) * (nb - min(nb, 3) + 1)).floor())
    mask = (seen * (1 << torch.arange(nb, device=d))).sum(1).to(torch.uint8)
    # the call's parameters: 2 % of each range around the truth, within the range
    par = torch.minimum(torch.maximum(truth + 0.02 * (hi - lo) * normal(10, n), torch.minimum(lo, truth)),
                        torch.maximum(hi, truth))
    dt = torch.float64 if case.get("prec") == "f64" else torch.float32
    s = dict(op=op, ctx=ctx, sfh=SFH[sfh], z=z.to(dt), par=par.to(dt).contiguous(), obs=obs, sigma=sigma.float(),
             mask=mask, prec=PREC[case.get("prec", "f32")], table="prec" not in case)
    if op.endswith("vjp"):
        s["gbar"] = normal(n, nb).float()
    if op in ("logpost", "hmc"):
        b = f64(BOUNDS)
        s["bounds"] = torch.cat([b, f64([[1.0, 0.0]] * 10)], 1).float().contiguous()
        s["prior"] = f64([[0.0, 1.5, 0.0]] * 10).float().contiguous()
        x = torch.logit(((par - b[:, :1]) / (b[:, 1:] - b[:, :1])).clamp(0.02, 0.98))
        if op == "hmc":   # chains that start near the mode, as after a search for it
            c = case["n_chain"]
            s["start"] = (x[None] + 0.05 * normal(c, 10, n)).float().contiguous()
            s["cfg"] = dict(n_chain=c, n_leapfrog=case["n_leapfrog"], n_warmup=case["n_warmup"],
                            n_sample=case["n_sample"], init_step=0.02, seed=seed)
        else:
            s["par"] = x.float().contiguous()
    return s


def run(s):
    ctx, op = s["ctx"], s["op"]
    if op in ("loglike", "exact_loglike"):
        logl, grad = ctx.loglike_grad(s["sfh"], s["par"], s["z"], s["obs"], s["sigma"], s["mask"],
                                      path=sps.SPS_PATH_APPROX if s["table"] else sps.SPS_PATH_EXACT, prec=s["prec"])
        return dict(logl=logl, grad=grad)
    if op == "logpost":
        logp, grad = ctx.logpost_grad(s["sfh"], s["par"], s["z"], s["obs"], s["sigma"], s["mask"], s["bounds"], s["prior"])
        return dict(logp=logp, grad=grad)
    if op == "mags":
        return dict(mag=ctx.phot_approx(s["sfh"], s["par"], s["z"]))
    if op == "exact_mags":
        return dict(mag=ctx.phot_exact(s["sfh"], s["par"], s["z"], prec=s["prec"]))
    if op == "hmc":
        return ctx.hmc_run(s["sfh"], s["z"], s["obs"], s["sigma"], s["mask"], s["bounds"], s["prior"], s["start"],
                           keep_samples=True, **s["cfg"])
    par = s["par"].detach().requires_grad_()
    mag = (sps.phot_approx(ctx, par, s["z"], sfh=s["sfh"]) if s["table"]
           else sps.phot_exact(ctx, par, s["z"], sfh=s["sfh"], prec=s["prec"]))
    grad, = torch.autograd.grad(mag, par, s["gbar"])
    return dict(mag=mag.detach(), grad=grad)


def work(case):
    n, nb, nw, op = case["n"], case["n_band"], n_wave_of(case), case["op"]
    grad = not op.endswith("mags")
    size = 8 if case.get("prec") == "f64" else 4
    per = size * 11 + (8 * nb + 1 if op in ("loglike", "logpost", "exact_loglike", "hmc") else 0)
    per += {"loglike": 44, "exact_loglike": 44, "logpost": 44, "hmc": 0}.get(op, size * nb + (40 + 4 * nb if grad else 0))
    if "prec" in case:
        # one matrix product over the wavelengths that a band reaches within 8 widths, one more for the gradient
        c = filters(nb)["center_A"]
        share = math.log10((c[-1] + 8 * SIGMA_A) / (c[0] - 8 * SIGMA_A)) / 3.0
        return dict(bytes=n * per + size * N_SSP * nw * share, flops=2.0 * n * N_SSP * nw * share * (2 if grad else 1))
    evals, out = n, n * per
    if op == "hmc":
        c, s = case["n_chain"], case["n_sample"]
        evals = n * c * (1 + case["n_leapfrog"] * (case["n_warmup"] + s))
        out = n * (per + 4 * (31 + c * (21 + 10 * s)))
    # the products with the two nodes of the z table around a galaxy, forward and adjoint
    return dict(bytes=out + 4.0 * min(N_Z, 2 * n) * nb * N_SSP, flops=evals * 4.0 * nb * N_SSP * (2 if grad else 1))


def exact(case, seed):
    op, n = case["op"], case["n"]
    if op == "hmc" or n > 200_000:   # a chain's accept steps have no value of their own; a sweep takes minutes
        return None
    s = prepare(case, seed)
    sfh, table, nb = case["sfh"], s["table"], case["n_band"]
    m = model(n_wave_of(case), nb, table)
    step = max(64, 512 if table else 512 * 1000 // n_wave_of(case))
    parts = []
    for i in range(0, n, step):
        q = slice(i, min(i + step, n))
        x, z = s["par"][:, q].double().requires_grad_(), s["z"][q].double()
        if op == "logpost":
            b, pr = s["bounds"].double(), s["prior"].double()
            th = b[:, :1] + (b[:, 1:2] - b[:, :1]) * torch.sigmoid(b[:, 2:3] * (x - b[:, 3:]))
        else:
            th = x
        mag = magnitudes(m, sfh, th, z, table)
        if op.endswith("mags"):
            parts.append(dict(mag=mag.detach()))
            continue
        if op.endswith("vjp"):
            grad, = torch.autograd.grad(mag, x, s["gbar"][q].double())
            parts.append(dict(mag=mag.detach(), grad=grad))
            continue
        sig = s["sigma"][q].double()
        lnp = -0.5 * ((mag - s["obs"][q].double()) / sig) ** 2 - torch.log(sig * math.sqrt(2 * math.pi))
        seen = (s["mask"][q, None].long() >> torch.arange(nb, device=z.device)) & 1
        val = (lnp * seen).sum(1)
        if op == "logpost":
            y = (x - pr[:, :1]) / pr[:, 1:2]
            val = val + (math.log(2.0) - torch.log(pr[:, 1:2]) - 0.5 * math.log(2 * math.pi) - 0.5 * y * y
                         + torch.special.log_ndtr(pr[:, 2:] * y)).sum(0)
        grad, = torch.autograd.grad(val.sum(), x)
        parts.append({"logp" if op == "logpost" else "logl": val.detach(), "grad": grad})
    return {k: torch.cat([p[k] for p in parts], 1 if k == "grad" else 0) for k in parts[0]}
