"""GPU: the batch kernel for many chunks (above 24 per compute unit) against the
one for few: the same packets, so the same counters and deposits (sums of n equal
terms in another order: n 2^-52; images: an FP32 rounding for each addition)."""
import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deposit_slots", [8, 16])
@pytest.mark.parametrize("chunks", [1, 2])  # beyond the limit: one more, twice as many
def test_both_kernels(chunks, deposit_slots):
    import torch
    limit = 24 * torch.cuda.get_device_properties(0).multi_processor_count
    packets = [chunks * limit - 1200, 700, 501]
    models = scenes.batch(len(packets), 4, 1.0, side=(8, 24))
    assert all(m.scene.n_lambda == 1 for m in models)
    runs = []
    for chunk in (1, 0):  # a chunk per packet; the few that the library takes
        ctx = mcrt.Context(0)
        sims = [mcrt.Sim(ctx, m.scene, mcrt.FP32, chunk=chunk, deposit_slots=deposit_slots) for m in models]
        res = [s.new_result() for s in sims]
        mcrt.batch_run_into(sims, res, packets, seed=11)
        runs.append([(r.stats(), r.table(), r.image(0), r.energy()) for r in res])
        for s in sims:
            s.close()
        ctx.close()
    eps = 2.0 ** -52
    for n, (sa, ta, ia, ea), (sb, tb, ib, eb) in zip(packets, *runs):
        assert all(sa[c] == sb[c] for c in sa if c != "kernel_ms") and sa["packets"] == n
        assert np.array_equal(ta != 0, tb != 0)
        assert np.allclose(ta, tb, rtol=(sa["packets"] + sa["events"]) * eps, atol=0)
        assert np.allclose(ea, eb, rtol=sa["prop_cells"] * eps, atol=1e-300)
        assert np.array_equal(ia != 0, ib != 0) and np.allclose(ia, ib, rtol=sa["peel_adds"] * 2.0 ** -23, atol=0)
