"""The coarsest level solved mode by mode is the result of its red-black
sweeps: a solve by one V(2,2) cycle over levels of 32^3 and 16^3 is compared
with the cycle in NumPy, for sweep counts on both sides of the rule that
chooses between the two kernels, with and without the mean projected out."""
from __future__ import annotations

import numpy as np
import pytest

from synth import uniform_particles

from helpers import lib_config, make_sim

pytestmark = pytest.mark.gpu


def _neighbours(e):
    return sum(np.roll(e, s, ax) for ax in range(3) for s in (1, -1))


def _sweeps(e, r, scale, kappa, count):
    """count red-black sweeps of (Lap e) / scale - kappa e = r."""
    parity = np.indices(r.shape).sum(0) & 1
    for _ in range(count):
        for colour in (0, 1):
            e = np.where(parity == colour, (_neighbours(e) - scale * r) / (6.0 + scale * kappa), e)
    return e


def _vcycle(r, kappa, count):
    e = _sweeps(np.zeros_like(r), r, 1.0, kappa, 2)
    t = r - (_neighbours(e) - (6.0 + kappa) * e)
    for ax in range(3):                          # full weighting
        t = 0.5 * t + 0.25 * (np.roll(t, 1, ax) + np.roll(t, -1, ax))
    c = t[::2, ::2, ::2]
    if kappa == 0.0:
        c = c - c.mean()
    c = _sweeps(np.zeros_like(c), c, 4.0, kappa, count)
    if kappa == 0.0:
        c -= c.mean()
    for ax in range(3):                          # trilinear
        c = np.stack([c, 0.5 * (c + np.roll(c, -1, ax))], ax + 1)
        c = c.reshape(c.shape[:ax] + (32,) + c.shape[ax + 2:])
    return _sweeps(e + c, r, 1.0, kappa, 2)


@pytest.mark.parametrize("coarse_sweeps", [1, 7, 8, 9, 33, 64])
@pytest.mark.parametrize("kappa", [0.0, 1e-4, 0.1])
@pytest.mark.parametrize("prec", [0, 1])
def test_one_cycle(coarse_sweeps, kappa, prec):
    ng, box, n = 32, 100.0, 2000
    x, p, ids = uniform_particles(n, box, 5)
    cfg = lib_config(ng, box, precision=prec, tol=0.99, n_initial=n, mg_levels=2,
                     coarse_sweeps=coarse_sweeps, cycles_per_outer=1)
    sim = make_sim(cfg, n)
    sim.bind(x, p, ids)
    sim.deposit()
    st = sim.solve(kappa, 1.0)
    assert st["vcycles"] == 1
    # fewer sweeps where they reduce the slowest mode 1e3-fold
    rho = 6.0 / (6.0 + 4.0 * kappa) if kappa else (4.0 + 2.0 * np.cos(2.0 * np.pi / 16)) / 6.0
    count = min(coarse_sweeps, int(np.ceil(np.log(1e-3) / (2.0 * np.log(rho)))))
    want = _vcycle(sim.rhs.cpu().numpy(), kappa, count)
    if kappa == 0.0:
        want -= want.mean()
    # each half sweep rounds 8 operations of its result, and passes what was
    # there on with a factor of at most one
    eps = 2.0**-24 if prec == 0 else 2.0**-53
    tol = 16 * (count + 4) * eps * np.abs(want).max()
    assert np.abs(sim.phi_numpy() - want).max() <= tol
    sim.close()
