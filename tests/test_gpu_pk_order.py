"""Power spectra of particles in random order, which are deposited block by
block, against the same particles in spatial order, which are not: the counts
are integers, so the meshes are equal, and the shells' sums differ by the order
in which their up to 2^20 positive terms are added (2^20 2^-53); one particle
in a wrong cell would change them by more than a millionth of the shot noise.
Sizes: the smallest that is ordered,
one that fills the sort's buffer to within a particle and one with a single
particle in the second part."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _points(n, box, seed):
    rng = np.random.default_rng(seed)
    x = rng.random((3, n)) * box
    half = n // 2
    x[:, :half] = (box * 0.37 + rng.normal(size=(3, half)) * 0.02 * box) % box
    x[:, 0] = 0.0
    x[:, 1] = np.nextafter(box, 0.0)
    return x


def _both(x, box, ng):
    import torch

    from paper_1709_04703_amd import power_spectrum

    order = np.lexsort((x[0] // (box / ng), x[1] // (box / ng * 8), x[2] // (box / ng * 8)))
    a = power_spectrum(torch.as_tensor(x, device="cuda"), box, ng)
    b = power_spectrum(torch.as_tensor(np.ascontiguousarray(x[:, order]), device="cuda"), box, ng)
    assert np.array_equal(a["modes"], b["modes"])
    assert np.abs(a["p_raw"] / b["p_raw"] - 1.0).max() <= 2.0**-33


@pytest.mark.parametrize("ng,n", [(128, (1 << 19) - 1), (128, 1 << 19), (128, 2_000_003), (128, 4_100_001),
                                  (256, 600_001)])
def test_random_order_equals_spatial_order(ng, n):
    _both(_points(n, 50.0, n), 50.0, ng)


def test_one_particle_in_the_last_part():
    # the buffer of 128^3 holds a fixed number of particles: walk n over it
    ng, box = 128, 50.0
    bytes_ = 2 * 16 * ng * ng * (ng // 2 + 1)
    fit = bytes_ // 17
    while True:
        chunks = -(-fit // 1024)
        tab = (chunks + 1) * 256
        need = (4 * fit + tab + -(-tab // 4096) + 1) * 4 + 1024 + 513 * 8
        if need <= bytes_:
            break
        fit -= fit // 64 + 1
    x = _points(fit + 1, box, 7)
    for n in (fit - 1, fit, fit + 1):
        _both(x[:, :n], box, ng)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -1e-9, 50.1])
def test_out_of_range_is_refused(bad):
    import torch

    import paper_1709_04703_amd as P

    x = _points(1 << 19, 50.0, 1)
    x[1, 400_000] = bad
    with pytest.raises(P.SdpmError, match="EDOMAIN"):
        P.power_spectrum(torch.as_tensor(x, device="cuda"), 50.0, 128)
