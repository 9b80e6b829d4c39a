"""GPU: the compaction of histories into training samples at the edges of its
tiles of 1024 records (events per packet from 1 to more than a tile, packets
that leave the last tile, or the only one, partly filled), against the records
compacted on the host."""
import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [mcrt.FP32, mcrt.FP64_VALIDATE])
@pytest.mark.parametrize("events,packets", [(1, 1), (1, 1023), (1, 1024), (1, 1025), (3, 341), (3, 342), (16, 64),
                                            (16, 65), (16, 70_000), (64, 33), (1000, 7), (1025, 9), (4096, 5)])
def test_samples_are_the_records(events, packets, precision):
    sc = scenes.sphere(n=8, tau=3.0, albedo=0.8, g=0.3, npix=8)
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, sc, precision)
    h = sim.collect(sim.new_result(), packets, seed=events, max_events=events)
    rec, tot = h.records()
    X, KP, C = h.samples()
    kind = np.float32 if precision == mcrt.FP32 else np.float64
    rec, tot = rec.astype(kind), tot.astype(kind)
    L = rec[:, :, 12]
    with np.errstate(divide="ignore", invalid="ignore"):
        want = np.where(L > 0, (tot[:, None] - rec[:, :, 13]) / np.where(L > 0, L, 1), 0).astype(np.float32)
    keep = want > 0
    assert h.n_samples == np.count_nonzero(keep) == len(C)
    assert np.array_equal(X, rec[keep][:, :9].astype(np.float32))
    assert np.array_equal(KP, rec[keep][:, 9:12].astype(np.float32))
    # one subtraction and one division in the run's precision
    assert np.allclose(C, want[keep], rtol=2.0 ** -22, atol=0)
    total = C.astype(np.float64).sum()
    assert abs(h.weight_sum - total) <= max(1, len(C)) * 2.0 ** -52 * total
    h.close()
    sim.close()
    ctx.close()
