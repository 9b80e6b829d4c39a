"""GPU: launches around the sizes where their shape changes (one chunk to a
wave, two waves to a SIMD, the queue; sums of direct light; copies): every
packet runs once, and the energy closes over the shards of the tallies."""
import dataclasses

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


def scene(kind, n_lambda):
    sc = scenes.disk((12, 11, 7), 1, 9) if kind == "disk" else scenes.sphere(12, 0.5, 0.5, 0.3)
    rep = lambda a: np.repeat(np.asarray(a, np.float64)[:1], n_lambda)
    return dataclasses.replace(sc, lambdas=0.5 + 0.01 * np.arange(n_lambda), kappa=rep(sc.kappa), albedo=rep(sc.albedo),
                               hg_g=rep(sc.hg_g), lum=1.0 + np.arange(n_lambda))


@pytest.mark.parametrize("precision", [mcrt.FP32, mcrt.FP64_VALIDATE])
@pytest.mark.parametrize("kind", ["disk", "sphere"])
@pytest.mark.parametrize("n_lambda", [1, 5])
def test_every_packet_once(n_lambda, kind, precision):
    sc = scene(kind, n_lambda)
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, sc, precision)
    res = sim.new_result()
    # 256 compute units: 2048, 3072 and 4096 waves; 12288 packets; 32 and 64 lanes to a wave
    edges = [1, 2, 2048, 3072, 4096, 12288, 32768, 65536, 196608]
    for total in sorted({max(1, e // n_lambda + d) for e in edges for d in (-1, 0, 1)}):
        res.zero()
        sim.run_into(res, total, seed=total)
        s, (emitted, absorbed, escaped, truncated) = res.stats(), res.energy()
        assert s["packets"] == total * n_lambda and s["peel_adds"] >= s["packets"]
        # a packet's L / n in the images' precision, summed in FP64
        rtol = 1e-6 if precision == mcrt.FP32 else 1e-10
        assert np.isclose(emitted, sc.lum.sum(), rtol=rtol, atol=0)
        assert np.isclose(absorbed + escaped + truncated, emitted, rtol=20 * rtol, atol=0)
        assert np.isclose(res.table().sum(), absorbed, rtol=1e-9, atol=0)
    again = res.energy(), res.stats()
    sim.run_into(res, total, seed=total)  # adds to what is there
    assert res.stats()["prop_cells"] == 2 * again[1]["prop_cells"]
    assert np.allclose(res.energy(), 2 * np.asarray(again[0]), rtol=1e-12, atol=1e-300)
    sim.close()
    ctx.close()
