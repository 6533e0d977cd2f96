"""The HMC kernel of large batches (k_hmc, two lanes per chain) and the line to the one of small batches
(k_hmc_pair, a pair of waves per chain)."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import MAX_EXCUSED, bounds_prior, dev, draws_follow_oracle, f32, gal_inputs

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


def first(args, m):
    """The arguments of the first m galaxies."""
    return [args[0], *(a[:m].contiguous() for a in args[1:5]), *args[5:7],
            None if args[7] is None else args[7][..., :m].contiguous()]


@pytest.mark.parametrize("start", ["given", "prior"])
@pytest.mark.parametrize("kind", ["dpl", "lognormal_burst"])
def test_both_kernels_draw_the_same_chains(ctx, kind, start):
    # a chain per galaxy, so that chain ids, and with them the draws, do not depend on the number of galaxies:
    # the same galaxies by either kernel, through warm-up with an adapted metric.  The kernels differ only in
    # the order of FP64 sums (1e-16), which moves the rounding of an FP32 value derived from one (6e-8) about
    # once in 1e8 values; ~100 values per evaluation, 97 evaluations, 8192 chains: less than one chain expected
    # to part by more than rounding, one in a thousand allowed
    m = PAIR_MAX[kind]
    args = problem(ctx, kind, 8200, 1, 883)
    if start == "prior":
        args[7] = None
    kw = dict(n_chain=1, n_leapfrog=4, n_warmup=20, n_sample=4, init_step=0.01, seed=5, adapt_metric=True,
              keep_samples=True)
    pairs, batched = ctx.hmc_run(*first(args, m), **kw), ctx.hmc_run(*args, **kw)
    same = torch.ones(m, dtype=torch.bool, device="cuda")
    for key in ("samples", "step", "inv_metric", "post_mean", "post_sd", "accept"):
        a, b = pairs[key], batched[key][..., :m]
        assert torch.isfinite(a).all() and torch.isfinite(b).all()
        same &= (a == b).reshape(-1, m).all(dim=0)
    assert (pairs["inv_metric"] != 1).any() and 0.3 < pairs["accept"].mean() < 1
    assert (~same).sum() <= m // 1000


@pytest.mark.parametrize("kind,adapt", [("dpl", True), ("lognormal_burst", False)])
def test_batched_kernel_split_and_blocked_runs(ctx, kind, adapt):
    # 1025 galaxies x 8 chains through the z-ordered chain state: the run split over three calls, and with other
    # numbers of iterations per launch, draws what one call draws
    n, C, n_w, n_s = 1025, 8, 20, 6
    args = problem(ctx, kind, n, C, 885)
    kw = dict(n_chain=C, n_leapfrog=2, n_warmup=n_w, n_sample=n_s, init_step=0.02, seed=6, adapt_metric=adapt)
    whole = ctx.hmc_run(*args, keep_samples=True, **kw)
    keys = ("post_mean", "post_sd", "rhat", "accept", "step", "inv_metric")
    state, smp = ctx.hmc_state(n, C), torch.zeros_like(whole["samples"])
    for b, e in ((0, 7), (7, 22), (22, n_w + n_s)):
        part = ctx.hmc_run(*args, it_begin=b, it_end=e, state=state, samples=smp, **kw)
    ctx.status()
    assert torch.equal(smp, whole["samples"]) and all(torch.equal(part[k], whole[k]) for k in keys)
    default = ctx.get_launch()
    for block in (1, 9):
        ctx.set_launch(hmc_block_iters=block)
        again = ctx.hmc_run(*args, keep_samples=True, **kw)
        assert torch.equal(again["samples"], whole["samples"]) and all(torch.equal(again[k], whole[k]) for k in keys)
    ctx.set_launch(**default)


@pytest.mark.parametrize("ctx", [6], indirect=True)      # the oracle's bands
def test_batched_kernel_log_normal_draws_follow_the_oracle(ctx, orc):
    n, C = 2050, 4
    args = problem(ctx, "lognormal_burst", n, C, 887)
    kw = dict(n_chain=C, n_leapfrog=10, n_warmup=1, n_sample=2, init_step=0.01, seed=404)
    out = ctx.hmc_run(*args, keep_samples=True, **kw)
    pick = np.random.default_rng(888).choice(n, 6, replace=False)
    host = [a.cpu().numpy().astype(np.float64) for a in args[1:4]]
    ref = orc.hmc_run(args[0], *(a[pick] for a in host), args[4].cpu().numpy()[pick], *bounds_prior(),
                      args[7].cpu().numpy().astype(np.float64).transpose(0, 2, 1)[:, pick], keep_samples=True,
                      keep_trace=True, gal_id=pick, n_gal_total=n, **kw)
    ok, excused = draws_follow_oracle(out["samples"].cpu().numpy()[..., pick].transpose(0, 1, 3, 2), ref)
    assert ok.all() and excused.mean() <= MAX_EXCUSED, (ok, excused)
