"""Exact-path calls at the ends of what they accept: a grid that ends short of a band."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import dev, gal_inputs, soa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec_name", ["SPS_F32", "SPS_BF16X"])
@pytest.mark.parametrize("n", [129, 400, 16384])     # ranked by one block, and by passes of their own
def test_band_past_the_end_of_the_grid(filt6, n, prec_name):
    # a grid from 3000 A: at z > 1.3 the bluest band lies more than 8 widths below its first wavelength, to
    # 13 widths its sums are still FP32 numbers.  Batches in z order leave bands out of a wave's reach out;
    # the same 100 galaxies in one row tile, never in z order, keep every term.  Where the band comes near
    # the grid the terms left out are at most 3e-9 of it; where it does not, none may be.  The same sums in
    # the same order within a tile of 128 wavelengths, the tiles' added in order: FP32 rounding of a
    # magnitude up to 128, 4e-6 each, of the sums, 1e-6 mag
    import paper_2506_19919_amd as sps
    prec = getattr(sps, prec_name)
    g = synth.ssp_grid(1500)
    k = g["wave_A"] >= 3000.0
    cut = dict(g, wave_A=g["wave_A"][k].copy(), lum=np.ascontiguousarray(g["lum"][..., k]))
    ctx = sps.Context(cut, filt6, precisions=(prec,), max_gal=n, max_exact=n)
    sfh, th, z = gal_inputs("dpl", 100, 861)
    at = np.arange(n) % 100
    few = ctx.phot_exact(sfh, soa(th), dev(z), prec=prec).cpu().numpy()
    many = ctx.phot_exact(sfh, soa(th[at]), dev(z[at]), prec=prec).cpu().numpy()
    ctx.close()
    blue = (3000.0 * (1 + z) - synth.filters()["center_A"][0]) / synth.filters()["sigma_A"][0]
    assert ((blue > 8) & (blue < 12)).sum() >= 5 and np.isfinite(few[blue < 12]).all()
    assert np.array_equal(np.isfinite(many), np.isfinite(few[at]))
    ok = np.isfinite(many)
    assert np.abs(many[ok] - few[at][ok]).max() <= 1e-5


@pytest.mark.parametrize("e", [-124, -118, -110, -40, 90])
def test_f32_keeps_its_precision_at_any_scale_of_the_grid(filt6, e):
    # SPS_F32 carries its operands as three BF16 parts, the last 16 bits below the first: a grid in small units
    # keeps all of them.  Magnitudes to the FP32 path's 1e-4 of the FP64 path on the same grid, and the
    # gradient, which no scale changes, to 1e-6 of the unscaled grid's largest component
    import paper_2506_19919_amd as sps
    n = 150
    sfh, th, z = gal_inputs("dpl", n, 871)
    gbar = dev(np.random.default_rng(872).normal(size=(n, 6)))
    base = synth.ssp_grid(500)
    grads = []
    for lum in (base["lum"], np.ldexp(base["lum"], e)):
        ctx = sps.Context(dict(base, lum=lum), filt6, precisions=(sps.SPS_F64, sps.SPS_F32), max_gal=n, max_exact=n)
        ref = ctx.phot_exact(sfh, soa(th, torch.float64), dev(z, torch.float64), prec=sps.SPS_F64)
        par = soa(th).requires_grad_()
        mag = sps.phot_exact(ctx, par, dev(z), sfh=sfh, prec=sps.SPS_F32)
        assert (mag.detach() - ref).abs().max() <= 1e-4
        grads.append(ctx.phot_vjp(sfh, soa(th), dev(z), gbar, path=sps.SPS_PATH_EXACT, prec=sps.SPS_F32))
        again, = torch.autograd.grad(mag, par, gbar)       # through the kept band sums
        assert (again - grads[-1]).abs().max() <= 1e-6 * grads[-1].abs().max()
        ctx.close()
    bar = 1e-6 * grads[0].abs().max(dim=0, keepdim=True).values
    assert ((grads[1] - grads[0]).abs() <= bar).all()


@pytest.mark.parametrize("prec_name", ["SPS_F32", "SPS_BF16X"])
@pytest.mark.parametrize("n_band,n", [(1, 400), (6, 129), (6, 4096), (6, 16384)])
def test_steep_attenuation_without_a_floor(ssp2000, n_band, n, prec_name):
    # exp(-tau_V x^delta) with delta = -3 (or 2) and no floor rises so fast across a blue band that the band's flux comes
    # from beyond 8 of its widths.  Batches in z order against the same 100 galaxies in one row tile, whose window and
    # sums leave nothing of them out; terms are only left out where they are below 1e-5 of the largest, and what
    # of them adds up stays under 5e-5 mag (FP32 rounding of a magnitude up to 256 included)
    import paper_2506_19919_amd as sps
    prec = getattr(sps, prec_name)
    ctx = sps.Context(ssp2000, synth.filters(n_band), precisions=(prec,), max_gal=n, max_exact=n)
    sfh, th, z = gal_inputs("dpl", 100, 881)
    r = np.random.default_rng(882)
    steep = r.random(100) < 0.3
    th[:, 7], th[:, 8], th[:, 9] = 4 * r.random(100), -1.5 * r.random(100), 0.3 * r.random(100) * (r.random(100) < 0.5)
    th[steep, 7], th[steep, 8], th[steep, 9] = r.uniform(1.5, 4, steep.sum()), -3.0, 0.0
    th[0, 7:], z[0] = (200.0, 2.0, 0.0), 1.65
    at = np.arange(n) % 100
    few = ctx.phot_exact(sfh, soa(th), dev(z), prec=prec).cpu().numpy()
    many = ctx.phot_exact(sfh, soa(th[at]), dev(z[at]), prec=prec).cpu().numpy()
    ctx.close()
    assert np.array_equal(np.isfinite(many), np.isfinite(few[at]))
    ok = np.isfinite(many) & (few[at] < 256)
    assert ok.mean() > 0.9 and np.abs(many[ok] - few[at][ok]).max() <= 5e-5
