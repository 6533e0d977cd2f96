"""The approximate path's kernels by batch size, against each other: the same galaxies in one call of
70,001 (a lane per galaxy, the form the FP64 oracle pins at full size) and in slices that take a pair of
waves, four lanes and two lanes per galaxy.

The pairs of waves take every FP32 sum in the one-lane order; only the FP64 total of the smooth mass
differs in its order (1e-16), which can move the rounding of FP32 values derived from it by one unit
(6e-8): within 2e-6 of a galaxy's largest gradient component, 2e-5 of log L's scale at the residuals used
here.  Four and two lanes add partial sums of 94 / G bins: up to 94 roundings of 6e-8 of terms that
cancel about tenfold in the shape parameters, 5e-5 of the largest component."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import bounds_prior, dev, f32, gal_inputs, soa

pytestmark = pytest.mark.gpu

PAIR_MAX, FOUR_MAX = 8192, 32768        # above them four, then (to 65,536) two, then one lane per galaxy
N = 70001
# a single galaxy, a ragged few and the most that pairs take; four lanes at both ends of their range; two
SLICES = [(0, 1), (1, 64), (64, 64 + PAIR_MAX), (8256, 8256 + PAIR_MAX + 1), (16449, 16449 + FOUR_MAX),
          (N - FOUR_MAX - 1, N)]


@pytest.fixture(scope="module", params=[1, 6, 8])
def ctx(request, ssp2000):
    import paper_2506_19919_amd as sps
    c = sps.Context(ssp2000, synth.filters(request.param), precisions=(sps.SPS_F64, sps.SPS_F32), max_gal=N)
    c.build_ztable(64, 0.1, 3.0)
    yield c
    c.close()


def batch(kind, nb):
    sfh, th, z = gal_inputs(kind, N, 811)
    z[[5, 70, 9000]] = [0.05, 3.5, 3.2]           # outside the table: NaN on both paths
    z[[6, 71]] = [0.1, 3.0]                       # its first and last node
    th[7, 4], th[72, 4] = 1.0, 0.0                # all burst, no burst
    th[8, 5], th[73, 5] = 11.5, 3.0               # a burst past every bin (empty window), below the grid
    rng = np.random.default_rng(812)
    obs, sig = f32(rng.uniform(20, 26, (N, nb))), f32(rng.uniform(0.3, 1.0, (N, nb)))
    mask = rng.integers(0, 1 << nb, N).astype(np.uint8)
    return sfh, f32(th), f32(z), obs, sig, mask


def close(a, b, rel):
    assert np.array_equal(np.isnan(a), np.isnan(b))
    scale = np.nan_to_num(np.abs(b)).max(axis=1, keepdims=True)
    assert np.all((np.abs(a - b) <= rel * np.maximum(scale, 1e-30)) | np.isnan(b))


@pytest.mark.parametrize("kind", ["dpl", "lognormal_burst"])
@pytest.mark.parametrize("op", ["mags", "loglike", "logl", "logpost", "vjp"])
def test_batch_sizes_agree(ctx, kind, op):
    nb = ctx.n_band
    sfh, th, z, obs, sig, mask = batch(kind, nb)
    if op == "logpost":
        bnd, pri = bounds_prior()
        th = f32((th - th.mean(0)) / (th.std(0) + 1e-3))      # unbounded values of order one
        bp = (dev(bnd), dev(pri))

    def call(lo, hi):
        t = lambda a: dev(np.ascontiguousarray(a[lo:hi]))
        p, zz, o, s, m = soa(th[lo:hi]), t(z), t(obs), t(sig), dev(mask[lo:hi], torch.uint8)
        if op == "mags":
            return [ctx.phot_approx(sfh, p, zz)]
        if op == "vjp":
            return [ctx.phot_vjp(sfh, p, zz, o).T]
        if op == "logl":
            return [ctx.loglike_grad(sfh, p, zz, o, s, m, grad=False)[:, None]]
        v, g = (ctx.logpost_grad(sfh, p, zz, o, s, m, *bp) if op == "logpost" else
                ctx.loglike_grad(sfh, p, zz, o, s, m))
        return [v[:, None], g.T]

    whole = [x.cpu().numpy().astype(np.float64) for x in call(0, N)]
    assert np.isnan(whole[0][[5, 70, 9000]]).all()
    for lo, hi in SLICES:
        for a, b in zip(call(lo, hi), whole):
            rel = 5e-5 if hi - lo > PAIR_MAX else 2e-6
            close(a.cpu().numpy().astype(np.float64), b[lo:hi], max(rel, 2e-5) if b.shape[1] == 1 else rel)
    with pytest.raises(Exception):
        ctx.status()                              # the redshifts outside the table were flagged


@pytest.mark.parametrize("n", [2048, 2050])
def test_hmc_at_the_limit_of_the_small_batch_kernel(ssp2000, filt6, orc, n):
    # 8192 chains: a pair of waves each; 8200: the batched kernel.  Both follow the oracle draw by draw
    import paper_2506_19919_amd as sps
    from gpu_common import MAX_EXCUSED, draws_follow_oracle
    C = 4
    ctx = sps.Context(ssp2000, filt6, max_gal=n * C)
    ctx.build_ztable(64, 0.1, 3.0)
    sfh, th, z = gal_inputs("dpl", n, 821)
    noise, sig = synth.photometric_noise(n, 6, 822)
    obs, sig = f32(orc.phot_approx(sfh, th, z) + noise), f32(sig)
    masks = synth.band_masks(n, 6, 823)
    bnd, pri = bounds_prior()
    frac = np.clip((th - bnd[:, 0]) / (bnd[:, 1] - bnd[:, 0]), 0.02, 0.98)
    x0 = f32(np.log(frac / (1 - frac))[None] + 0.05 * np.random.default_rng(824).normal(size=(C, n, 10)))
    kw = dict(n_chain=C, n_leapfrog=3, n_warmup=0, n_sample=2, init_step=0.01, seed=407)
    out = ctx.hmc_run(sfh, dev(z), dev(obs), dev(sig), dev(masks, torch.uint8), dev(bnd), dev(pri),
                      dev(np.ascontiguousarray(np.transpose(x0, (0, 2, 1)))), keep_samples=True, **kw)
    ref = orc.hmc_run(sfh, z, obs, sig, masks, bnd, pri, x0, keep_samples=True, keep_trace=True, **kw)
    ok, excused = draws_follow_oracle(out["samples"].cpu().numpy().transpose(0, 1, 3, 2), ref)
    assert ok.all() and excused.mean() <= MAX_EXCUSED
    ctx.close()
