"""The log-normal bins' rules against the FP64 oracle: narrow widths, whose old bins take the closed
form, to wide ones, whose bins stay with the nodes, at peaks on both sides of the observation time.
Seven galaxies take the two-wave kernel, 8193 the kernel of four lanes per galaxy (the same galaxies
repeated in random order, so that lanes of one wave take different rules)."""
import numpy as np
import pytest

from gpu_common import dev, f32, gal_inputs, soa
from test_gpu_vjp import _gbar, _ref, ctx, vjp_ok  # noqa: F401  (ctx: the module's fixture)


def grid():
    w, tp, z = [a.ravel() for a in np.meshgrid([0.2, 0.21, 0.3, 0.5, 0.75, 1.0, 1.5], [1.0, 3.0, 6.0, 12.0],
                                               [0.1, 1.1, 2.95], indexing="ij")]
    sfh, th, _ = gal_inputs("lognormal_burst", w.size, 901)
    th[:, 1], th[:, 2] = tp, w
    return sfh, f32(th), f32(z)


@pytest.mark.gpu
def test_weights(ctx, orc):
    # every weight to 1e-4 (|x| dx with |x| <= 13 and FP32 x, ~1e-6 / w), or 1e-7 of the mass formed
    sfh, th, z = grid()
    w, ref = ctx.weights(sfh, soa(th), dev(z)).cpu().numpy().astype(np.float64), orc.weights(sfh, th, z)
    for g in range(z.size):
        np.testing.assert_allclose(w[g], ref[g], rtol=1e-4, atol=1e-7 * 10 ** th[g, 0])


@pytest.mark.gpu
@pytest.mark.parametrize("n", [7, 8193])
def test_vjp(ctx, orc, n):
    import paper_2506_19919_amd as sps
    sfh, th, z = grid()
    at = np.random.default_rng(902).integers(0, z.size, n)
    gbar = _gbar(z.size, 903)
    g = ctx.phot_vjp(sfh, soa(th[at]), dev(z[at]), dev(gbar[at]), path=sps.SPS_PATH_APPROX).cpu().numpy().T
    ref, absref = _ref(orc, sfh, th, z, gbar, 0)
    assert vjp_ok(g, ref[at], absref[at]).all()
