"""One V-cycle against the same cycle in NumPy, to rounding: every way in which
a level is smoothed, restricted and prolonged (fused passes, tiles, separate
kernels for other sweep counts) gives the textbook cycle."""
from __future__ import annotations

import numpy as np
import pytest

from synth import uniform_particles

from helpers import lib_config, make_sim

pytestmark = pytest.mark.gpu


def _neighbours(e):
    return sum(np.roll(e, s, ax) for ax in range(3) for s in (1, -1))


def _sweeps(e, r, scale, kappa, count):
    parity = np.indices(r.shape).sum(0) & 1
    for _ in range(count):
        for colour in (0, 1):
            e = np.where(parity == colour, (_neighbours(e) - scale * r) / (6.0 + scale * kappa), e)
    return e


def _vcycle(r, kappa, level, levels, pre, post, coarse_sweeps):
    scale = 4.0**level
    e = np.zeros_like(r)
    if level == levels - 1:
        n = r.shape[0]
        rho = 6.0 / (6.0 + scale * kappa) if kappa else (4.0 + 2.0 * np.cos(2.0 * np.pi / n)) / 6.0
        count = min(coarse_sweeps, int(np.ceil(np.log(1e-3) / (2.0 * np.log(rho)))))
        if kappa == 0.0:
            r = r - r.mean()
        e = _sweeps(e, r, scale, kappa, count)
        return e - e.mean() if kappa == 0.0 else e
    e = _sweeps(e, r, scale, kappa, pre)
    t = r - (_neighbours(e) - 6.0 * e) / scale + kappa * e
    for ax in range(3):                          # full weighting
        t = 0.5 * t + 0.25 * (np.roll(t, 1, ax) + np.roll(t, -1, ax))
    c = _vcycle(t[::2, ::2, ::2], kappa, level + 1, levels, pre, post, coarse_sweeps)
    for ax in range(3):                          # trilinear
        c = np.stack([c, 0.5 * (c + np.roll(c, -1, ax))], ax + 1)
        c = c.reshape(c.shape[:ax] + (-1,) + c.shape[ax + 2:])
    return _sweeps(e + c, r, scale, kappa, post)


CASES = [(ng, levels, pre, post, kappa)
         for ng, levels in ((16, 2), (32, 3), (64, 3), (128, 4))
         for pre, post in ((2, 2), (1, 1), (3, 2)) for kappa in (0.0, 1e-4)]
# the NumPy cycle takes long at this size
CASES += [(256, 5, 2, 2, 1e-4), (256, 5, 3, 2, 1e-4)]


@pytest.mark.parametrize("ng,levels,pre,post,kappa", CASES)
@pytest.mark.parametrize("prec", [0, 1])
def test_one_cycle(ng, levels, pre, post, kappa, prec):
    box, n = 100.0, 3000
    x, p, ids = uniform_particles(n, box, ng)
    cfg = lib_config(ng, box, precision=prec, tol=0.99, n_initial=n, mg_levels=levels, pre=pre,
                     post=post, cycles_per_outer=1)
    sim = make_sim(cfg, n)
    sim.bind(x, p, ids)
    sim.deposit()
    st = sim.solve(kappa, 1.0)
    assert st["vcycles"] == 1
    want = _vcycle(sim.rhs.cpu().numpy(), kappa, 0, levels, pre, post, cfg.coarse_sweeps)
    if kappa == 0.0:
        want -= want.mean()
    # every half sweep rounds 8 operations of its result and passes what was
    # there on with a factor of at most one
    eps = 2.0**-24 if prec == 0 else 2.0**-53
    tol = 16 * (cfg.coarse_sweeps + levels * (pre + post)) * eps * np.abs(want).max()
    assert np.abs(sim.phi_numpy() - want).max() <= tol
    sim.close()


# no sweep after the prolongation, which then adds to both colours of what the
# pre-smoothing left: on meshes with a second correction array and without
@pytest.mark.parametrize("ng,levels", [(64, 3), (128, 4), (256, 5)])
@pytest.mark.parametrize("prec", [0, 1])
def test_one_cycle_without_post_smoothing(ng, levels, prec):
    test_one_cycle(ng, levels, 2, 0, 1e-4, prec)


# From 2^25 cells on, FP32 levels outside V(2,2) form the residual apart from
# its restriction: the same cycle, so it converges as on the next smaller mesh,
# whose residual is restricted as it is formed.
@pytest.mark.parametrize("pre,post", [(1, 1), (3, 3), (2, 0)])
def test_cycles_do_not_depend_on_the_mesh(pre, post):
    import torch

    kappa, tol, cycles = 0.05, 1e-7, []
    for ng in (256, 512):
        box, n = 100.0, 3000
        x, p, ids = uniform_particles(n, box, 1)
        cfg = lib_config(ng, box, precision=0, tol=tol, n_initial=n, pre=pre, post=post)
        sim = make_sim(cfg, n)
        sim.bind(x, p, ids)
        sim.deposit()
        cycles.append(sim.solve(kappa, 1.0)["vcycles"])
        phi = sim.phi
        lap = sum(torch.roll(phi, s, d) for d in range(3) for s in (1, -1)) - 6.0 * phi
        res = (lap.sub_(phi, alpha=kappa)).sub_(sim.rhs)
        assert float(res.norm()) <= 1.01 * tol * float(sim.rhs.norm())
        sim.close()
        del sim, phi, lap, res
        torch.cuda.empty_cache()
    assert cycles[1] <= cycles[0] + 1
