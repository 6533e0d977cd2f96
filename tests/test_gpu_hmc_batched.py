"""The HMC kernel of large batches (k_hmc, two lanes per chain) and the line to the one of small batches
(k_hmc_pair, a pair of waves per chain)."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import bounds_prior, dev, f32, gal_inputs

pytestmark = pytest.mark.gpu

PAIR_MAX = {"dpl": 6144, "lognormal_burst": 8192}     # most chains that a pair of waves each takes


@pytest.fixture(scope="module", params=[1, 6])
def ctx(request, ssp2000):
    import paper_2506_19919_amd as sps
    c = sps.Context(ssp2000, synth.filters(request.param), precisions=(sps.SPS_F64,), max_gal=1 << 14)
    c.build_ztable(64, 0.1, 3.0)
    yield c
    c.close()


def problem(ctx, kind, n, C, seed, z=None):
    """hmc_run's arguments for n galaxies x C chains that start near the truth."""
    sfh, th, zz = gal_inputs(kind, n, seed)
    th[:, 3] = np.maximum(th[:, 3], 0.5)
    th[:, synth.P_FFLOOR] = np.maximum(th[:, synth.P_FFLOOR], 0.02)
    zz = zz if z is None else np.full(n, z)
    p, zd = dev(th.T), dev(f32(zz))
    nb = ctx.n_band
    obs = ctx.phot_approx(sfh, p, zd) + 0.05 * dev(np.random.default_rng(seed).normal(size=(n, nb)))
    mask = dev(np.random.default_rng(seed + 1).integers(1, 1 << nb, n), torch.uint8)
    bnd, pri = bounds_prior()
    frac = np.clip((th - bnd[:, 0]) / (bnd[:, 1] - bnd[:, 0]), 0.02, 0.98)
    x0 = np.log(frac / (1 - frac)).T[None] + 0.05 * np.random.default_rng(seed + 2).normal(size=(C, 10, n))
    return [sfh, zd, obs, torch.full_like(obs, 0.1), mask, dev(bnd), dev(pri), dev(x0)]


@pytest.mark.parametrize("kind", ["dpl", "lognormal_burst"])
@pytest.mark.parametrize("z", [None, 1.0])
def test_the_line_between_the_kernels_costs_nothing(ctx, kind, z):
    # eight more chains, and the kernel of large batches, must not be the faster call: within 8 % of each
    # other's best time of several in turn (repeats differ by 1 to 2 %).  Also at 8192 chains, where the lines
    # of the kernels were once drawn alike
    for n in {PAIR_MAX[kind], 8192}:
        best = {}
        args = {m: problem(ctx, kind, m, 1, 881, z) for m in (n, n + 8)}
        for rep in range(8):
            for m in (n, n + 8):
                t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                t0.record()
                ctx.hmc_run(*args[m], n_chain=1, n_leapfrog=10, n_warmup=1, n_sample=2, init_step=0.01, seed=3)
                t1.record()
                t1.synchronize()
                best[m] = min(best.get(m, 1e9), t0.elapsed_time(t1)) if rep else 1e9
        assert best[n] <= 1.08 * best[n + 8], (n, best)
