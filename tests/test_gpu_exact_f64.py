"""The FP64 exact path at the edges of its tiles (32 galaxies x 16 wavelengths, one or two wavelength
tiles at a time, several per block) against the FP64 oracle: sums of 1128 weights and up to 2000
wavelengths in another order agree to 1e-12 mag, so the bound is the weights' (closed forms 1e-9 mag, the
double power law's quadrature 1e-8)."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import dev, gal_inputs, soa

MAG_TOL = {"dpl": 1e-8, "lognormal": 1e-9}


@pytest.mark.gpu
@pytest.mark.parametrize("n_wave,n_band,ns", [(2000, 6, (1, 31, 32, 33, 64, 65)), (500, 1, (16, 97, 513)),
                                              (1001, 8, (33, 161, 1500, 4500))])
def test_f64_tiles(oracle_mod, n_wave, n_band, ns):
    import paper_2506_19919_amd as sps
    ssp, filt = synth.ssp_grid(n_wave), synth.filters(n_band)
    orc = oracle_mod.Oracle(ssp, filt)
    ctx = sps.Context(ssp, filt, precisions=(sps.SPS_F64,), max_gal=max(ns), max_exact=max(ns))
    for n in ns:
        for kind in MAG_TOL:
            sfh, th, z = gal_inputs(kind, n, 1300 + n)
            z[n // 2] = 0.1
            m = ctx.phot_exact(sfh, soa(th, torch.float64), dev(z, torch.float64), prec=sps.SPS_F64).cpu().numpy()
            pick = np.unique(np.r_[0, n // 2, n - 1, np.random.default_rng(n).integers(0, n, 20)])
            ref = orc.phot_exact(sfh, th[pick], z[pick])
            assert np.abs(m[pick] - ref).max() <= MAG_TOL[kind], (n, kind, np.abs(m[pick] - ref).max())
    ctx.close()
