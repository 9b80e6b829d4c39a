"""GPU: copies between the device and ordinary arrays at the edges of their
ways (a result small enough for pinned memory, one below and at the size from
which copies go in chunks, a last chunk that is not full, more chunks than
slots), and from two threads at once.  All ways move or scale the same bits."""
import ctypes
import threading

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt, scenes

pytestmark = pytest.mark.gpu


def on_device(res, j):
    """The image as the kernel writes it to a device buffer."""
    import torch
    out = torch.full(res.sim.image_shapes[j], -1.0, dtype=torch.float64, device="cuda")
    mcrt._check(mcrt.lib().mcrt_result_image(res.h, j, ctypes.c_void_p(out.data_ptr()), out.numel()))
    return out.cpu().numpy()


@pytest.mark.parametrize("precision", [mcrt.FP32, mcrt.FP64_VALIDATE])
@pytest.mark.parametrize("npix", [1, 64, 65, 89, 91, 127, 129, 256, 363, 727, 1031])
def test_images(npix, precision):
    sc = scenes.disk((9, 7, 5), 2, npix)
    ctx = mcrt.Context(0)
    sim = mcrt.Sim(ctx, sc, precision)
    res = sim.run(3000, seed=5)
    for j in range(len(sim.image_shapes)):
        a, b = res.image(j), on_device(res, j)
        assert a.shape == b.shape and np.count_nonzero(a) > 0 and np.array_equal(a, b)
        # the SED is the sum of the image (another order, 2 npix^2 terms of one sign)
        assert np.allclose(res.sed(j), a.sum(axis=(1, 2)), rtol=1e-12, atol=0)
    sim.close()
    ctx.close()


@pytest.mark.parametrize("n", [1, 29127, 29128, 131_072, 140_001])
def test_network_copies(n):
    """9 n floats in, 40 n out, in chunks or not: rows as in slices that are
    too small for chunks."""
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, 9)).astype(np.float32)
    ctx = mcrt.Context(0)
    p = mcrt.Proposal(ctx, seed=3)
    whole = p.forward(X)
    for lo in range(0, n, 6400):
        assert np.array_equal(whole[lo:lo + 6400], p.forward(X[lo:lo + 6400]))
    p.close()
    ctx.close()


def test_two_threads():
    """Each thread reads its own results while the other copies."""
    ctx = mcrt.Context(0)
    jobs = []
    for seed in (1, 2):
        sim = mcrt.Sim(ctx, scenes.disk((9, 7, 5), 4, 700 + seed))
        res = sim.run(2000, seed=seed)
        jobs.append((sim, res, [on_device(res, j) for j in range(len(sim.image_shapes))]))
    bad = []

    def read(res, want):
        for _ in range(10):
            for j, w in enumerate(want):
                if not np.array_equal(res.image(j), w):
                    bad.append(j)
            res.stats(), res.energy(), res.sed(0)

    threads = [threading.Thread(target=read, args=(res, want)) for _, res, want in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for sim, _, _ in jobs:
        sim.close()
    ctx.close()
