"""The re-sort at sizes where its passes split differently: fewer particles
than a wavefront, a workgroup's keys and the scan's segments with a remainder,
and both sides of the size from which a lane takes sixteen keys; particles
spread over the mesh and all in one cell.  Against NumPy's stable sort."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import lib_config, make_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 63, 65, 1023, 1025, 4097, 300_001, (1 << 21) - 1, 1 << 21,
                               (1 << 21) + 4097])
@pytest.mark.parametrize("spread", [True, False])
@pytest.mark.parametrize("prec", [0, 1])
def test_sort(n, spread, prec):
    ng, box, shift = 64, 64.0, 4
    rng = np.random.default_rng(n)
    x = rng.random((n, 3)) * box if spread else 20.25 + 0.5 * rng.random((n, 3))
    p = np.arange(3 * n, dtype=np.float64).reshape(n, 3) % 1000.0
    ids = np.arange(n, dtype=np.uint32)
    cfg = lib_config(ng, box, precision=prec, sort_every=1, sort_shift=shift, n_initial=n)
    sim = make_sim(cfg, n)
    sim.bind(x, p, ids)
    sim.sort()
    gx, gp, gid = sim.particles()
    cell = np.floor(x).astype(np.int64)
    key = np.zeros(n, dtype=np.int64)
    for b in range(2):
        for d in range(3):
            key |= ((cell[:, d] >> shift >> b) & 1) << (3 * b + d)
    key = key << 8 | (cell[:, 2] & 15) << 4 | (cell[:, 1] & 15)
    want = np.argsort(key, kind="stable")
    assert np.array_equal(gid, ids[want])
    assert np.array_equal(gx, x[want])
    assert np.array_equal(gp, p[want])
    sim.close()
