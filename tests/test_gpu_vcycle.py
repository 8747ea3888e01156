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


def _box_vcycle(r, kappa, level, boxes, pre, post, coarse_sweeps):
    """The cycle on a frozen-exterior box: boxes[l] = (lo, hi) in (x, y, z) of
    level l, everything 0 outside them."""
    def inside(n, box):
        m = np.zeros((n, n, n), dtype=bool)
        m[tuple(slice(box[0][d], box[1][d] + 1) for d in (2, 1, 0))] = True
        return m

    def sweeps(e, count):
        for _ in range(count):
            for colour in (0, 1):
                e = np.where(box & (parity == colour),
                             (_neighbours(e) - scale * r) / (6.0 + scale * kappa), e)
        return e

    n, scale = r.shape[0], 4.0**level
    box, parity = inside(n, boxes[level]), np.indices(r.shape).sum(0) & 1
    e = np.zeros_like(r)
    if level == len(boxes) - 1:
        return sweeps(e, min(coarse_sweeps, _sweeps_for_1e3(boxes[level], level, kappa)))
    e = sweeps(e, pre)
    t = np.where(box, r - (_neighbours(e) - 6.0 * e) / scale + kappa * e, 0.0)
    for ax in range(3):
        t = 0.5 * t + 0.25 * (np.roll(t, 1, ax) + np.roll(t, -1, ax))
    c = _box_vcycle(t[::2, ::2, ::2], kappa, level + 1, boxes, pre, post, coarse_sweeps)
    for ax in range(3):
        c = np.stack([c, 0.5 * (c + np.roll(c, -1, ax))], ax + 1)
        c = c.reshape(c.shape[:ax] + (-1,) + c.shape[ax + 2:])
    return sweeps(np.where(box, e + c, 0.0), post)


def _sweeps_for_1e3(box, level, kappa):
    rho = (sum(2.0 * np.cos(np.pi / (hi - lo + 2)) for lo, hi in zip(*box)) /
           (6.0 + 4.0**level * kappa))
    return max(1, int(np.ceil(np.log(1e-3) / (2.0 * np.log(rho)))))


# boxes whose faces lie anywhere in the tiles, columns and vectors of the passes
@pytest.mark.parametrize("ng,levels,radius,pre,post",
                         [(ng, levels, radius, pre, post)
                          for ng, levels, radii in ((32, 3, (6.2, 9.7)), (64, 4, (9.4, 22.6)),
                                                    (128, 5, (30.3, 53.8)))
                          for radius in radii for pre, post in ((2, 2), (1, 1), (3, 2), (2, 0))] +
                         [(256, 5, 90.7, 2, 2), (256, 5, 101.2, 2, 1)])
@pytest.mark.parametrize("kappa", [0.02, 0.4])
@pytest.mark.parametrize("prec", [0, 1])
def test_one_cycle_on_a_box(ng, levels, radius, pre, post, kappa, prec):
    box, n = 10.0 * ng, 3000
    rng = np.random.default_rng(ng)
    # off the mesh's centre, so that the faces differ from axis to axis
    obs = (0.5 * box + 4.0, 0.5 * box - 13.0, 0.5 * box + 21.0)
    x = np.array(obs) + rng.uniform(-20.0, 20.0, size=(n, 3))
    cfg = lib_config(ng, box, c_grav=-1.0, shrink=1, precision=prec, tol=0.99, n_initial=n,
                     mg_levels=levels, pre=pre, post=post, cycles_per_outer=1, box_align=1, x_obs=obs)
    sim = make_sim(cfg, n)
    sim.bind(x, np.zeros((n, 3)), np.arange(n))
    sim.shrink_radius(radius * box / ng)
    st = sim.state()
    assert st["periodic"] == 0
    # the levels' boxes, down to the first that its own sweeps solve
    boxes = [(list(st["lo"]), list(st["hi"]))]
    for level in range(1, levels):
        lo, hi = boxes[-1]
        lo, hi = [(v + 1) >> 1 for v in lo], [min(v >> 1, (ng >> level) - 2) for v in hi]
        if any(b < a for a, b in zip(lo, hi)):
            break
        boxes.append((lo, hi))
        if level < levels - 1 and _sweeps_for_1e3(boxes[-1], level, kappa) <= pre + post + 1:
            break
    sim.deposit()
    assert sim.solve(kappa, 1.0)["vcycles"] == 1
    got, rhs = sim.phi_numpy(), np.zeros((ng,) * 3)
    sl = tuple(slice(st["lo"][d], st["hi"][d] + 1) for d in (2, 1, 0))
    rhs[sl] = sim.rhs.cpu().numpy()[sl]
    want = _box_vcycle(rhs, kappa, 0, boxes, pre, post, cfg.coarse_sweeps)
    eps = 2.0**-24 if prec == 0 else 2.0**-53
    tol = 16 * (cfg.coarse_sweeps + levels * (pre + post)) * eps * np.abs(want).max()
    assert np.abs(got - want).max() <= tol
    sim.close()
