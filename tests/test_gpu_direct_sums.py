"""GPU: the FP64 sums of direct light up to their largest launch.  Without
dust every packet adds the same value to one pixel per wavelength.  Tolerance:
the value's own roundings (L / n, the phase function, the product: at most 4),
a wave's share (6 additions of a tree over 64 lanes) and the pixel's one
addition, half a unit in the last place each."""
import dataclasses

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_lambda", [1, 3])
@pytest.mark.parametrize("packets", [5, 8193, 16_384, 32_767, 32_768])
def test_direct_sums(packets, n_lambda):
    one = np.ones(n_lambda)
    sc = dataclasses.replace(scenes.sphere(n=9, npix=15, albedo=0.0, incl_deg=20.0), lambdas=0.5 * (1 + np.arange(n_lambda)),
                             kappa=0 * one, albedo=0 * one, hg_g=0 * one, lum=0.7 + np.arange(n_lambda))
    ctx = mcrt.Context(0)
    a, b = [mcrt.Sim(ctx, sc, prec) for prec in (mcrt.FP32, mcrt.FP64_VALIDATE)]
    ra, rb = a.run(packets, seed=3), b.run(packets, seed=3)
    x, y = ra.image(0), rb.image(0)
    assert np.array_equal(x != 0, y != 0) and np.count_nonzero(y) == n_lambda
    assert np.all(np.abs(x - y) <= (4 + 6 + 1) * 2.0 ** -24 * y)
    assert ra.stats()["peel_adds"] == packets * n_lambda
    for s in (a, b):
        s.close()
    ctx.close()
