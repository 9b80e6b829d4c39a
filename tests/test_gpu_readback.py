"""GPU: the table's readback at the edges of its tiles (wavelengths below, at
and above a tile's 64, odd grids, bricks cut by the grid, a destination on the
device or on the host, a host readback in several passes)."""
import dataclasses

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


def disk(n, n_lambda):
    sc = scenes.disk(n, 2, 8)
    lam = scenes.log_lambdas(n_lambda) if n_lambda > 1 else np.array([0.55])
    kappa, albedo, g = scenes.powerlaw_optics(lam, 1.0, 0.6)
    return dataclasses.replace(sc, lambdas=lam, kappa=kappa, albedo=np.zeros(n_lambda), hg_g=g,
                               lum=1.0 + np.arange(n_lambda) / n_lambda)


def tables(sc, packets, **tune):
    import torch
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, sc, mcrt.FP64_VALIDATE, **tune)
    res = sim.run(packets, seed=2)
    host = res.table()
    dev = torch.full((sim.n_cells, sim.n_lambda), -1.0, dtype=torch.float64, device="cuda")
    res.table(out=dev)
    absorbed = res.energy()[1]
    sim.close()
    ctx.close()
    assert np.array_equal(host, dev.cpu().numpy())
    assert abs(host.sum() - absorbed) <= 1e-10 * absorbed
    return host


@pytest.mark.parametrize("n_lambda", [1, 2, 3, 63, 64, 65, 130])
@pytest.mark.parametrize("n", [(7, 5, 3), (33, 17, 9), (64, 32, 16)])
def test_table_layouts_agree(n, n_lambda):
    """The same packets with other storage bricks: the same table in natural
    order (FP64 sums of the same deposits in another order: 1e-12)."""
    sc = disk(n, n_lambda)
    a = tables(sc, 200)
    for brick in ((0, 0, 5), (5, 0, 0), (1, 3, 1)):
        b = tables(sc, 200, brick=brick)
        assert np.array_equal(a != 0, b != 0) and np.allclose(a, b, rtol=1e-12, atol=0)


def test_octree_readback():
    sc = scenes.torus(5, 4, 67, 8, n_clumps=25, tau_eq=8.0)
    assert np.count_nonzero(tables(sc, 50)) > 0


def test_host_readback_in_passes():
    """More than 2^25 elements go to the host in several passes."""
    sc = disk((8, 8, 8), 70_000)
    t = tables(sc, 1)
    assert np.count_nonzero(t.sum(axis=0)) > 60_000 and np.count_nonzero(t[-8:]) + np.count_nonzero(t[:8]) > 0


@pytest.mark.parametrize("npix", [1, 127, 128, 129, 300])
def test_sed_parts(npix):
    """SED = sum of the image's pixels (FP64 sums of up to 9e4 values: 1e-12)."""
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, scenes.disk((16, 16, 8), 3, npix), mcrt.FP32)
    res = sim.run(2000, seed=1)
    for j in range(3):
        assert np.allclose(res.sed(j), res.image(j).sum(axis=(1, 2)), rtol=1e-12, atol=0)
    sim.close()
    ctx.close()
