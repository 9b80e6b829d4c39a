"""GPU: a result takes device memory for the copies that its launches add to
and for no more."""
import dataclasses

import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


# cells per axis, packets that pay for the copies (a 128-byte line each), copies with the table itself
@pytest.mark.parametrize("n,packets,copies", [(130, 650_000, 4), (165, 650_000, 2)])
def test_copies_memory(n, packets, copies):
    import torch
    sc = dataclasses.replace(scenes.sphere(n=n, npix=8, albedo=0.0), albedo=[0.0])
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, sc, mcrt.FP64_VALIDATE)
    res = sim.new_result()
    sim.run_into(res, 1000, seed=1)  # too few for copies
    res.stats()
    before = torch.cuda.mem_get_info()[0]
    sim.run_into(res, packets, seed=2)
    took = before - torch.cuda.mem_get_info()[0]
    # cells are stored in whole bricks, at most 8 cells long; 4 MB: the allocator's granularity
    assert (copies - 1) * 8 * n ** 3 <= took <= (copies - 1) * 8 * (n + 7) ** 3 + (4 << 20)
    assert res.stats()["packets"] == packets + 1000
    sim.close()
    ctx.close()
