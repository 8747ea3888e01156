"""Weight and bias gradients of a convolution layer at the sizes where the
matrix-core kernel's tiles change: rows shorter than one product (16), one
product (32), one and two workgroups per row (64, 128)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import conv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [16, 32, 64, 128])
def test_wgrad_against_fp64(n):
    import torch

    import paper_1709_04703_amd as P

    rng = np.random.Generator(np.random.PCG64(n))
    x = conv.bf16_round(np.maximum(rng.normal(size=(n, n, n, 16)), 0.0))
    g = conv.bf16_round(rng.normal(size=(n, n, n, 16)))

    def dev(a):
        return torch.as_tensor(a.astype(np.float32)).to("cuda:0").bfloat16().view(torch.int16)

    dw = torch.empty(27 * 256, dtype=torch.float32, device="cuda:0")
    db = torch.empty(16, dtype=torch.float32, device="cuda:0")
    scratch = torch.zeros(P.net_scratch_bytes(n), dtype=torch.uint8, device="cuda:0")
    P.conv3d_wgrad(n, dev(x), dev(g), dw, db, scratch)
    rw, rb, _ = conv.conv_wgrad(x, g)
    mw, mb, _ = conv.conv_wgrad(np.abs(x), np.abs(g))
    # the products of two BF16 values are exact in FP32; a sum of m of them in
    # any order is within gamma_m of the sum of their magnitudes, and no
    # workgroup's chain, reduction included, is longer than n^3 / 8 terms
    u = 2.0 ** -24
    m = n ** 3 / 8
    gamma = m * u / (1.0 - m * u)
    assert np.all(np.abs(dw.cpu().numpy().reshape(27, 16, 16) - rw) <= gamma * mw)
    assert np.all(np.abs(db.cpu().numpy() - rb) <= gamma * mb)
    # and in the norm far below the worst case (random signs: sqrt of the chain)
    assert np.linalg.norm(dw.cpu().numpy().reshape(27, 16, 16) - rw) <= 4 * np.sqrt(m) * u * np.linalg.norm(mw)


def test_wgrad_infinity_stays_in_its_products():
    """An infinite input value meets only the gradients its taps pair it with:
    with g zero around it except one voxel, one tap is infinite and no entry is
    NaN where the direct sum has none."""
    import torch

    import paper_1709_04703_amd as P

    n = 16
    x = np.zeros((n, n, n, 16))
    g = np.ones((n, n, n, 16))
    x[0, 0, 0, 3] = np.inf
    dw = torch.empty(27 * 256, dtype=torch.float32, device="cuda:0")
    db = torch.empty(16, dtype=torch.float32, device="cuda:0")
    scratch = torch.zeros(P.net_scratch_bytes(n), dtype=torch.uint8, device="cuda:0")

    def dev(a):
        return torch.as_tensor(a.astype(np.float32)).to("cuda:0").bfloat16().view(torch.int16)

    P.conv3d_wgrad(n, dev(x), dev(g), dw, db, scratch)
    got = dw.cpu().numpy().reshape(27, 16, 16)
    assert np.all(np.isinf(got[:, 3, :])) and np.all(got[:, 3, :] > 0)
    assert np.all(got[:, [c for c in range(16) if c != 3], :] == 0.0)
    assert np.all(db.cpu().numpy() == n ** 3)
