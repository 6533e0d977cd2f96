"""Exact-path batches ranked by one block (129 .. 16,383 galaxies) and the sizes around: magnitudes
against the FP64 path, which keeps the caller's order, and gradients against the same galaxies
evaluated in slices of one row tile, which is never ranked."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import dev, f32, gal_inputs, soa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_z", [0, 64, 1024])      # no z table (64 + 1 buckets), the usual one, the largest
@pytest.mark.parametrize("n", [128, 129, 1000, 16383, 16384])
def test_ranked_batches(filt6, n_z, n):
    import paper_2506_19919_amd as sps
    ssp = synth.ssp_grid(500)                       # 500 wavelengths: a ragged last tile
    ctx = sps.Context(ssp, filt6, precisions=(sps.SPS_F64, sps.SPS_F32, sps.SPS_BF16X), max_gal=n, max_exact=n)
    if n_z:
        ctx.build_ztable(n_z, 0.1, 3.0)
    sfh, th, z = gal_inputs("dpl", n, 841)
    z[3] = 3.7                                      # past the table: the overflow bucket, a valid exact galaxy
    th, z = f32(th), f32(z)
    ref = ctx.phot_exact(sfh, soa(th, torch.float64), dev(z, torch.float64), prec=sps.SPS_F64).cpu().numpy()
    zq = z.copy()
    zq[n // 2] = np.nan                             # a NaN redshift: NaN for that galaxy only
    rng = np.random.default_rng(842)
    gbar = f32(rng.normal(size=(n, 6)))
    ok = np.arange(n) != n // 2
    for prec, tol in ((sps.SPS_F32, 1e-4), (sps.SPS_BF16X, 2e-3)):
        m = ctx.phot_exact(sfh, soa(th), dev(zq), prec=prec).cpu().numpy()
        assert np.isnan(m[n // 2]).all()
        assert np.abs(m[ok] - ref[ok]).max() <= tol
        g = ctx.phot_vjp(sfh, soa(th), dev(zq), dev(gbar), path=sps.SPS_PATH_EXACT, prec=prec).cpu().numpy().T
        assert np.isnan(g[n // 2]).any() and np.isfinite(g[ok]).all()
        # slices of 100: the same sums over other windows and K ranges.  FP32 sums of ~1e3 terms: 1e-5 of
        # the largest component for FP32; BF16X's operands carry 2^-17 each: 1e-4
        for a in (0, (n // 100) * 100 - 100):
            s = slice(a, a + 100)
            gs = ctx.phot_vjp(sfh, soa(th[s]), dev(zq[s]), dev(gbar[s]), path=sps.SPS_PATH_EXACT, prec=prec)
            gs = gs.cpu().numpy().T
            k = ok[s]
            bar = (1e-5 if prec == sps.SPS_F32 else 1e-4) * np.abs(gs[k]).max(axis=1, keepdims=True)
            assert np.all(np.abs(g[s][k] - gs[k]) <= bar)
    ctx.close()
