"""GPU: results read into pinned host memory arrive whole, whatever their size,
and large ones by one copy of the device, not through other pinned memory and
the calling thread (which takes twice as long or more, as long as into ordinary
memory)."""
import ctypes
import statistics
import time

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


def pinned(shape, dtype):
    import torch
    return torch.zeros(shape, dtype=dtype, pin_memory=True)


def address(t):
    return ctypes.c_void_p(t.data_ptr())


@pytest.mark.parametrize("precision", [mcrt.FP32, mcrt.FP64_VALIDATE])
@pytest.mark.parametrize("npix", [5, 89, 91, 300])  # at most and above 64 KB, above 128 KB and 1 MB
def test_images(npix, precision):
    import torch
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, scenes.disk((9, 7, 5), 2, npix), precision)
    res = sim.run(2000, seed=3)
    for j in range(len(sim.image_shapes)):
        out, sed = pinned(sim.image_shapes[j], torch.float64), pinned((2,), torch.float64)
        mcrt._check(mcrt.lib().mcrt_result_image(res.h, j, address(out), out.numel()))
        mcrt._check(mcrt.lib().mcrt_result_sed(res.h, j, address(sed), 2))
        assert np.array_equal(out.numpy(), res.image(j)) and np.array_equal(sed.numpy(), res.sed(j))
    sim.close()
    ctx.close()


def test_table_and_network():
    import torch
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, scenes.disk((100, 100, 100), 4, 8), mcrt.FP32)
    res = sim.run(2000, seed=3)
    out, host = pinned((10 ** 6, 4), torch.float64), np.zeros((10 ** 6, 4))

    def read(p):
        t = time.perf_counter()
        mcrt._check(mcrt.lib().mcrt_result_absorption(res.h, p, host.size))
        return time.perf_counter() - t

    times = [(read(address(out)), read(ctypes.c_void_p(host.ctypes.data))) for _ in range(15)]
    assert np.array_equal(out.numpy(), host) and host.any()
    fast, slow = (statistics.median(t[k] for t in times) for k in (0, 1))  # 0.6 and 1.5 ms
    assert fast < 0.85 * slow
    p = mcrt.Proposal(ctx, seed=1)
    X = np.random.default_rng(1).normal(size=(30_000, 9)).astype(np.float32)
    O = pinned((30_000, 40), torch.float32)
    mcrt._check(mcrt.lib().mcrt_proposal_forward(p.h, X.ctypes.data, 30_000, address(O)))
    assert np.array_equal(O.numpy(), p.forward(X))
    p.close()
    sim.close()
    ctx.close()
