"""The layer kernel where its split of the mesh changes: masked data gradient
with 8 rows per workgroup (64) and with 4 (128), forward with more planes per
workgroup than its loop is unrolled by (128)."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import conv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,backward", [(64, True), (128, True), (128, False)])
def test_layer_against_fp64(n, backward):
    import torch

    import paper_1709_04703_amd as P

    rng = np.random.Generator(np.random.PCG64(n + backward))
    x = conv.bf16_round(rng.normal(size=(n, n, n, 16)))
    mask = conv.bf16_round(np.maximum(rng.normal(size=(n, n, n, 16)), 0.0))
    w = rng.normal(size=(27, 16, 16)) * 0.1
    b = rng.normal(size=16) * 0.1

    def dev(a):
        return torch.as_tensor(a.astype(np.float32)).to("cuda:0").bfloat16().view(torch.int16)

    out = torch.zeros((n**3, 16), dtype=torch.int16, device="cuda:0")
    wt = torch.as_tensor(w.astype(np.float32)).to("cuda:0")
    wq = conv.bf16_round(w)
    if backward:
        P.conv3d(n, dev(x), wt, None, P.CONV_BACKWARD_DATA | P.CONV_MASK, dev(mask), out)
        ref = conv.conv_dgrad(x, wq) * (mask > 0)
    else:
        P.conv3d(n, dev(x), wt, torch.as_tensor(b.astype(np.float32)).to("cuda:0"), P.CONV_RELU,
                 None, out)
        ref = np.maximum(conv.conv(x, wq, b), 0.0)
    got = out.view(torch.bfloat16).float().cpu().numpy().astype(np.float64).reshape(ref.shape)
    # the FP32 sum of 432 exact products and the bias is within gamma_433 of
    # the sum of magnitudes (|x| < 8 and |w| < 1 here), then one BF16 rounding
    u = 2.0 ** -24
    near = 433 * u * (conv.conv(np.abs(x), np.abs(wq), np.abs(b)) if not backward
                      else conv.conv_dgrad(np.abs(x), np.abs(wq)))
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 1.01 * near)
