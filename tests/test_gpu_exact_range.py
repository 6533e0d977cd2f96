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


@pytest.mark.parametrize("prec_name", ["SPS_F32", "SPS_BF16X"])
@pytest.mark.parametrize("grid,n_band,n", [("end", 6, 100), ("end", 1, 400), ("end", 6, 16384), ("gap", 6, 400)])
def test_gradient_of_a_band_past_the_end_of_the_grid(filt6, grid, n_band, n, prec_name):
    # bands of which the grid, from 3000 A or without 2500 .. 6000 A, holds only terms from 5 to 12 widths away: the
    # gradient with respect to the star formation and metallicity slots is made of the same terms as the magnitude.
    # Against the oracle's Jacobian to 1e-3, the bar of a gradient, of the sum of the bands' shares; galaxies whose
    # bands all lie within 12 widths, beyond which sums leave the FP32 range
    import paper_2506_19919_amd as sps
    from oracle import Oracle
    prec = getattr(sps, prec_name)
    g = synth.ssp_grid(1500)
    w = g["wave_A"]
    k = w >= 3000.0 if grid == "end" else (w < 2500.0) | (w >= 6000.0)
    cut = dict(g, wave_A=w[k].copy(), lum=np.ascontiguousarray(g["lum"][..., k]))
    filt = dict(center_A=filt6["center_A"][:n_band].copy(), sigma_A=filt6["sigma_A"][:n_band].copy())
    sfh, th, z = gal_inputs("dpl", 100, 891)
    gbar = np.random.default_rng(892).normal(size=(100, n_band))
    _, jac = Oracle(cut, filt).mags_jacobian(sfh, th.astype(np.float32), z.astype(np.float32), path=1)
    ref = np.einsum("gb,gbp->gp", gbar.astype(np.float32), jac)
    share = np.einsum("gb,gbp->gp", np.abs(gbar), np.abs(jac))[:, 1:7].max(1, keepdims=True)
    rest = (1 + z)[:, None, None] * w[k]
    width = np.abs((rest - filt["center_A"][:, None]) / filt["sigma_A"][:, None]).min(2).max(1)
    assert ((width > 8.2) & (width < 12)).sum() >= (5 if grid == "end" else 1) and ((width > 5) & (width < 8)).sum() >= 5
    ctx = sps.Context(cut, filt, precisions=(prec,), max_gal=n, max_exact=n)
    at = np.arange(n) % 100
    grad = ctx.phot_vjp(sfh, soa(th[at]), dev(z[at]), dev(gbar[at]), path=sps.SPS_PATH_EXACT, prec=prec).T.cpu().numpy()
    ctx.close()
    err = (np.abs(grad - ref[at]) / share[at])[:, 1:7].max(1)
    assert err[width[at] < 12].max() <= 1e-3
