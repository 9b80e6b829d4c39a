"""GPU: the loss adds a sample's weight times its negative log-likelihood with
one rounding.  Only one sample has a weight, and the same lane meets it in each
of three passes of the workgroups, so the loss is that lane's sum: exactly
round(w y + round(w y + round(w y))) in FP32, where y is the sample's own loss
(weight 1)."""
import numpy as np
import pytest

from paper_1705_04702_amd import mcrt

pytestmark = pytest.mark.gpu


def test_one_rounding():
    import torch
    n = 64 * 2 * torch.cuda.get_device_properties(0).multi_processor_count  # one pass of all workgroups
    rng = np.random.default_rng(4)
    ctx = mcrt.Context(0)
    p = mcrt.Proposal(ctx, seed=1)
    tell = 0
    for c in np.float32([1, 3, 5, 6, 7, 11, 13, 25, 0.7, 0.9, 1.3, 2.6]):
        X = rng.normal(size=(n, 9)).astype(np.float32)
        KP = rng.normal(size=(n, 3))
        KP = (KP / np.linalg.norm(KP, axis=1, keepdims=True)).astype(np.float32)
        i = int(rng.integers(n))
        y = np.float32(p.grad(X[i:i + 1], KP[i:i + 1], np.float32([1.0]))[0])
        C = np.zeros(n, np.float32)
        C[i] = c
        loss = p.grad(np.tile(X, (3, 1)), np.tile(KP, (3, 1)), np.tile(C, 3))[0]
        w = c * np.float32(1.0 / (3 * float(c)))
        wy = float(w) * float(y)  # exact, as are the sums below before they are rounded
        r = [np.float32(wy)]
        for _ in range(2):
            r.append(np.float32(wy + float(r[-1])))
        assert loss == float(r[2])
        tell += r[2] != np.float32(float(r[0]) * 3)  # the product rounded first gives something else
    assert tell > 0
    p.close()
    ctx.close()
