"""GPU: inputs in pinned host memory that an earlier copy on the context's
stream still fills are taken in their turn on the stream."""
import ctypes

import numpy as np
import pytest

from paper_1705_04702_amd import mcrt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1000, 29_128, 200_000])  # below, at and above the size that is copied in chunks
def test_input_filled_on_the_stream(n):
    import torch
    rng = np.random.default_rng(n)
    X = rng.normal(size=(n, 9)).astype(np.float32)
    KP = rng.normal(size=(n, 3))
    KP = (KP / np.linalg.norm(KP, axis=1, keepdims=True)).astype(np.float32)
    C = rng.exponential(1.0, n).astype(np.float32)
    ctx = mcrt.Context(0)
    p = mcrt.Proposal(ctx, seed=3)
    out, (loss, grad) = p.forward(X), p.grad(X, KP, C)
    busy = torch.randn(8192, 8192, device="cuda")
    on_device = torch.from_numpy(X).cuda()
    pinned = torch.zeros((n, 9), dtype=torch.float32, pin_memory=True)
    got, g, l = np.empty((n, 40), np.float32), np.empty(mcrt.MLP_PARAMS, np.float32), ctypes.c_double()
    address = ctypes.c_void_p(pinned.data_ptr())

    def fill():
        pinned.zero_()
        torch.cuda.synchronize()
        for _ in range(8):  # some milliseconds before the copy
            torch.mm(busy, busy)
        pinned.copy_(on_device, non_blocking=True)

    fill()
    mcrt._check(mcrt.lib().mcrt_proposal_forward(p.h, address, n, got.ctypes.data))
    assert np.array_equal(got, out)
    fill()
    mcrt._check(mcrt.lib().mcrt_proposal_grad(p.h, address, KP.ctypes.data, C.ctypes.data, n, ctypes.byref(l),
                                              g.ctypes.data))
    assert l.value == loss and np.array_equal(g, grad)
    p.close()
    ctx.close()
