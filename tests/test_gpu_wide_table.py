"""GPU: tables around 2^32 elements, where an element's number no longer fits
the 32 bits of a deposit slot: the FP32 run's deposits (through the slots)
against the FP64 run's (straight to the table), per wavelength and in place."""
import dataclasses

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["sphere", "disk"])
@pytest.mark.parametrize("n_lambda", [255, 256])  # times 2^24 cells: the last table of 32 bits, the first beyond
def test_deposits_in_place(n_lambda, kind):
    import torch
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GB of free device memory")
    side = (256, 256, 256)
    sc = scenes.sphere(n=256, npix=4) if kind == "sphere" else \
        dataclasses.replace(scenes.disk(side, 1, 4), instruments=scenes.disk((8, 8, 8), 1, 4).instruments[:1])
    rep = lambda a: np.repeat(np.asarray(a, np.float64)[:1], n_lambda)
    sc = dataclasses.replace(sc, lambdas=0.5 + 0.01 * np.arange(n_lambda), kappa=rep(sc.kappa), albedo=rep(sc.albedo),
                             hg_g=rep(sc.hg_g), lum=1.0 + np.arange(n_lambda))
    tables = []
    for precision in (mcrt.FP32, mcrt.FP64_VALIDATE):
        ctx = mcrt.Context(0)
        sim = mcrt.Sim(ctx, sc, precision)
        res = sim.run(300, seed=7)
        t = torch.empty((256 ** 3, n_lambda), dtype=torch.float64, device="cuda")
        tables.append((res.table(out=t), res.energy()[1]))
        sim.close()
        ctx.close()
    (a, ea), (b, eb) = tables
    step = 1 << 20  # cells at a time
    sums, off, norm = np.zeros((2, n_lambda)), 0.0, 0.0
    for c in range(0, 256 ** 3, step):
        x, y = a[c:c + step], b[c:c + step]
        sums += np.stack([x.sum(0).cpu().numpy(), y.sum(0).cpu().numpy()])
        off += float(((x - y) ** 2).sum())
        norm += float((y ** 2).sum())
    assert np.isclose(sums[0].sum(), ea, rtol=1e-9) and np.isclose(sums[1].sum(), eb, rtol=1e-9)
    # FP32 arithmetic: a packet of 300 may take another path at a threshold; a
    # misplaced wavelength or cell would be off by the whole of its deposits
    assert np.allclose(sums[0], sums[1], rtol=2e-2, atol=0) and off <= 0.05 ** 2 * norm
    del tables, t, a, b, x, y
    torch.cuda.empty_cache()
