"""GPU: batches of few chunks (models of few packets in small chunks, marching
apart; others draining apart) against the same batch in fixed chunks and in so
many chunks that the other kernel runs: the same packets, so the same counters
and deposits (sums of n equal terms in another order: n 2^-52)."""
import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [mcrt.FP32, mcrt.FP64_VALIDATE])
@pytest.mark.parametrize("packets", [[1], [1, 63, 64, 65], [3072, 3073], [5, 3071, 20_000, 257], [700] * 9])
def test_same_packets(packets, precision):
    models = scenes.batch(len(packets), 4, 1.0, side=(8, 24))
    runs = []
    for chunk in (0, 256, 2):
        ctx = mcrt.Context(0)
        sims = [mcrt.Sim(ctx, m.scene, precision, chunk=chunk) for m in models]
        res = [s.new_result() for s in sims]
        mcrt.batch_run_into(sims, res, packets, seed=11)
        runs.append([(r.stats(), r.table(), r.image(0), r.energy()) for r in res])
        for s in sims:
            s.close()
        ctx.close()
    for other in runs[1:]:
        for n, (sa, ta, ia, ea), (sb, tb, ib, eb) in zip(packets, runs[0], other):
            assert all(sa[c] == sb[c] for c in sa if c != "kernel_ms") and sa["packets"] == n
            eps = 2.0 ** -52
            assert np.array_equal(ta != 0, tb != 0)
            assert np.allclose(ta, tb, rtol=(sa["packets"] + sa["events"]) * eps, atol=0)
            assert np.allclose(ea, eb, rtol=sa["prop_cells"] * eps, atol=1e-300)
            unit = 2.0 ** -23 if precision == mcrt.FP32 else eps
            assert np.array_equal(ia != 0, ib != 0) and np.allclose(ia, ib, rtol=sa["peel_adds"] * unit, atol=0)
