"""GPU: launches on both sides of the queue's rules (packets per wave, FP64 sums
of the direct light, mixed or separate march loops), against the FP64
validation run of the same packets.

With albedo 0 a point source's image is its direct light: every packet adds
the same value to one pixel per wavelength.  Tolerance of that pixel: FP32
rounding of the optical depth, at most (n + 3) 2^-24 tau over the n < 100
cells of the ray (tau < 2 here), of its exponential, and of the additions: one
where the waves sum in FP64, else at most one per 32 packets, each at most
half a unit in the last place of the sum."""
import dataclasses

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


def scene(kind):
    if kind == "octree":
        sc = scenes.torus(max_depth=4, torus_depth=4, n_lambda=3, npix=16, tau_eq=1.0)
        return dataclasses.replace(sc, source="point_iso", albedo=np.zeros(3))
    sc = scenes.sphere(n=12, npix=15, albedo=0.0, incl_deg=20.0)
    if kind == "lambdas":
        return dataclasses.replace(sc, lambdas=np.array([0.5, 1.0, 2.0]), kappa=np.array([1.0, 0.5, 0.0]),
                                   albedo=np.zeros(3), hg_g=np.zeros(3), lum=np.array([1.0, 0.0, 3.0]))
    return sc


@pytest.mark.parametrize("kind", ["sphere", "lambdas", "octree"])
@pytest.mark.parametrize("packets", [1, 65, 4097, 8192, 8193, 140_000, 270_000])
def test_direct_light(kind, packets):
    sc = scene(kind)
    ctx = mcrt.Context(0)
    runs = {}
    for prec in (mcrt.FP32, mcrt.FP64_VALIDATE):
        sim = mcrt.Sim(ctx, sc, prec)
        res = sim.new_result()
        for half in ((0, packets // 2), (packets // 2, packets - packets // 2)):  # sums cleared between launches
            sim.run_into(res, packets, seed=9, first_id=half[0], count=half[1])
        sim.run_into(res, packets, seed=9)
        runs[prec] = (res.image(0), res.energy(), res.stats(), float(res.table().sum()))
        sim.close()
    ctx.close()
    (a, ea, sa, ta), (b, eb, sb, tb) = runs[mcrt.FP32], runs[mcrt.FP64_VALIDATE]
    assert sa["packets"] == sb["packets"] == 2 * packets * sc.n_lambda
    assert sa["events"] == sb["events"] == 0 and sa["peel_adds"] == sb["peel_adds"]
    assert np.array_equal(a != 0, b != 0) and np.count_nonzero(b) == np.count_nonzero(sc.lum)
    tol = (100 + 3 + 4) * 2.0 ** -24 * 2.0 + (4 if packets <= 8192 else 2 * packets / 32 + 4) * 2.0 ** -24
    nz = b != 0
    assert np.all(np.abs(a[nz] - b[nz]) <= tol * b[nz])
    assert np.allclose(ea, eb, rtol=1e-5, atol=1e-6 * eb[0])
    assert abs(ta - tb) <= 1e-5 * tb + 1e-300


@pytest.mark.parametrize("kind", ["disk", "disk64", "octree"])
def test_copies_merge(kind):
    """A launch long enough for further copies of its table (point source) or
    images (disk) equals the same packets in launches too short for them.
    Tables: FP64 sums of the same FP32 deposits, 1e-12.  The disk's images: the
    same FP32 values in another order; k additions to a pixel differ by at most
    k 2^-24 of it, and its brightest pixel gets fewer than 1700 (1e-4)."""
    if kind == "octree":
        sc = dataclasses.replace(scene("octree"), albedo=np.full(3, 0.4))
    else:
        sc = scenes.disk((19, 13, 7), 3, 21)
    n = 24_000 if kind != "disk64" else 22_500  # times 3 wavelengths: above 65536
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, sc, mcrt.FP64_VALIDATE if kind == "disk64" else mcrt.FP32)
    one, parts = sim.new_result(), sim.new_result()
    for _ in range(2):  # copies are clear again after a launch
        sim.run_into(one, n, seed=4)
        for k in range(3):
            sim.run_into(parts, n, seed=4, first_id=k * n // 3, count=n // 3)
    assert {k: v for k, v in one.stats().items() if k != "kernel_ms"} == \
        {k: v for k, v in parts.stats().items() if k != "kernel_ms"}
    a, b = one.table(), parts.table()
    assert np.array_equal(a != 0, b != 0) and np.allclose(a, b, rtol=1e-12, atol=0)
    for x, y in zip(one.images(), parts.images()) if kind != "octree" else ():
        assert np.array_equal(x != 0, y != 0) and np.allclose(x, y, rtol=1e-4, atol=0)
    sim.close()
    ctx.close()
