"""The exact path's backward from the forward's band sums against the one that forms them itself
(pinned to the FP64 oracle elsewhere), below and above the batch size from which the galaxies are put in
z order by passes of their own, in a single row tile and ragged ones.

Both take the same steps on the same band sums; the sums differ only where a batch's z order differs
between two calls (a large batch's order within a z bucket is free), by the rounding of up to 16 tile
sums of positive terms (1e-6), and the adjoint carries that to 1e-5 of a galaxy's largest component."""
import numpy as np
import pytest
import torch

from gpu_common import dev, gal_inputs, soa

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(ssp2000, filt6):
    import paper_2506_19919_amd as sps
    c = sps.Context(ssp2000, filt6, precisions=(sps.SPS_F32, sps.SPS_BF16X), max_gal=1 << 15, max_exact=1 << 15)
    c.build_ztable(64, 0.1, 3.0)
    yield c
    c.close()


@pytest.mark.parametrize("prec_name", ["SPS_F32", "SPS_BF16X"])
@pytest.mark.parametrize("kind,n", [("dpl", 1), ("lognormal_burst", 128), ("dpl", 129), ("dpl", 16383), ("dpl", 16384),
                                    ("lognormal_burst", 20011)])
def test_backward_from_band_sums(ctx, prec_name, kind, n):
    import paper_2506_19919_amd as sps
    prec = getattr(sps, prec_name)
    sfh, th, z = gal_inputs(kind, n, 1500 + n)
    par, zt = soa(th).requires_grad_(), dev(z)
    gbar = dev(np.random.default_rng(n).normal(0, 1, (n, 6)))
    mag = sps.phot_exact(ctx, par, zt, sfh=sfh, prec=prec)
    other = soa(np.roll(th, 1, axis=0))                    # a call in between: nothing is kept in the context
    ctx.phot_exact(sfh, other, zt, prec=prec)
    g1, = torch.autograd.grad(mag, par, gbar, retain_graph=True)
    g2, = torch.autograd.grad(mag, par, 2 * gbar)
    with torch.no_grad():
        plain = sps.phot_exact(ctx, par, zt, sfh=sfh, prec=prec)
    ref = ctx.phot_vjp(sfh, par.detach(), zt, gbar, path=sps.SPS_PATH_EXACT, prec=prec)
    assert (mag - plain).abs().max() <= 4e-6               # two units of an FP32 magnitude near 25
    bar = 1e-5 * ref.abs().max(dim=0, keepdim=True).values
    assert ((g1 - ref).abs() <= bar).all() and ((0.5 * g2 - ref).abs() <= bar).all()
