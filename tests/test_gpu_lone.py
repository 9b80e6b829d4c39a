"""GPU: marches that a whole wave takes for one packet (one packet to a wave)
against marches of full waves: the same packets, so the same counters and the
same deposits.  Sums of n equal terms in another order differ by n 2^-52 at
most; a march deposits once in a cell, and a packet marches once more than it
scatters."""
import dataclasses

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu

N = 1024
COUNTS = ("packets", "events", "prop_cells", "locate_cells", "peel_cells", "peel_adds", "peel_dropped", "capped")


def scene(n, kind, tau):
    if kind == "disk":
        return scenes.disk(n, 2, 16)
    sc = scenes.uniform_cube(1, tau0=tau, albedo=0.6, g=0.4)
    cells = int(np.prod(n))
    rho = np.random.default_rng(cells).random(cells).astype(np.float32)
    rho[:: 7] = 0.0  # empty cells
    return dataclasses.replace(sc, n=n, density=rho * sc.density.max())


def compare(sc, precision):
    ctx = mcrt.Context(0)
    full = mcrt.Sim(ctx, sc, precision, waves_per_cu=1)
    lone = mcrt.Sim(ctx, sc, precision)
    a = full.run(64 * N, seed=9)
    b = lone.new_result()
    for lo in range(0, 64 * N, N):  # fewer packets than waves: one to a wave
        lone.run_into(b, 64 * N, seed=9, first_id=lo, count=N)
    sa, sb = a.stats(), b.stats()
    assert [sa[c] for c in COUNTS] == [sb[c] for c in COUNTS] and sa["prop_cells"] > 0
    ta, tb = a.table(), b.table()
    eps = 2.0 ** -52
    assert np.array_equal(ta != 0, tb != 0)
    assert np.allclose(ta, tb, rtol=(sa["packets"] + sa["events"]) * eps, atol=0)
    assert np.allclose(a.energy(), b.energy(), rtol=sa["prop_cells"] * eps, atol=1e-300)
    for j in range(len(full.image_shapes)):
        x, y = a.image(j), b.image(j)
        # FP32: about 1e5 additions to the brightest pixel, each rounded to 2^-24
        rtol = 5e-3 if precision == mcrt.FP32 else sa["peel_adds"] * eps
        assert np.array_equal(x != 0, y != 0) and np.allclose(x, y, rtol=rtol, atol=0)
    for s in (full, lone):
        s.close()
    ctx.close()


@pytest.mark.parametrize("precision", [mcrt.FP32, mcrt.FP64_VALIDATE])
@pytest.mark.parametrize("n", [(1, 1, 1), (2, 1, 3), (21, 22, 20), (61, 45, 27), (3, 200, 5), (64, 64, 64)])
@pytest.mark.parametrize("kind,tau", [("disk", 0.0), ("cube", 0.5), ("cube", 20.0)])
def test_lone_packets(kind, tau, n, precision):
    compare(scene(n, kind, tau), precision)
