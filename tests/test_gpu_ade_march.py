"""The ADE sweep where its split over workgroups and lanes changes: the
smallest mesh, planes that do not fill the last workgroup, rows of one to eight
cells per lane with a ragged end, and sweeps that follow each other on the same
scratch.  Each cell's own update equation fixes the result: earlier neighbours
new, later ones old."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import ade

from helpers import lib_config, make_sim

pytestmark = pytest.mark.gpu


def _box_residual(old, new, f, lam, lo, hi, forward):
    """Largest |(1 + 3 lam) new - (1 - 3 lam) old - lam (S6 - f)| over the box;
    outside it old and new are the same frozen values."""
    sl = [slice(lo[d], hi[d] + 1) for d in (2, 1, 0)]
    s = 0.0
    for ax in range(3):
        for step in (-1, 1):
            nb = list(sl)
            nb[ax] = slice(sl[ax].start + step, sl[ax].stop + step)
            s = s + ((new if (step < 0) == forward else old)[tuple(nb)])
    c = tuple(sl)
    return np.abs((1 + 3 * lam) * new[c] - (1 - 3 * lam) * old[c] - lam * (s - f[c])).max()


@pytest.mark.parametrize("forward", [True, False])
def test_smallest_periodic_mesh(forward):
    ng, lam = 8, 8.8
    rng = np.random.default_rng(1)
    old, f = rng.normal(size=(ng,) * 3), rng.normal(size=(ng,) * 3)
    cfg = lib_config(ng, 100.0, c_grav=-1.0, precision=0, n_initial=1, solver=1)
    sim = make_sim(cfg, 1)
    sim.bind([[50.0, 50.0, 50.0]], [[0.0, 0.0, 0.0]], [0], phi=old)
    import torch

    sim.rhs.copy_(torch.as_tensor(f))
    sim.ade_sweep(lam, forward)
    sim.ade_sweep(lam, not forward)          # again on the scratch of the first
    ref = ade.sweep(old, f, lam, (0,) * 3, (ng - 1,) * 3, True, forward)
    ref = ade.sweep(ref, f, lam, (0,) * 3, (ng - 1,) * 3, True, not forward)
    assert np.abs(sim.phi_numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
    sim.close()


# cells of the box per axis: below, at and above the workgroup's 6 planes; two,
# four and eight cells per lane
@pytest.mark.parametrize("ng,cells", [(32, 5), (32, 7), (64, 13), (128, 71), (256, 135), (512, 263)])
@pytest.mark.parametrize("forward", [True, False])
def test_ragged_boxes(ng, cells, forward):
    import torch

    box, lam = 10.0 * ng, 8.8
    h = box / ng
    cfg = lib_config(ng, box, c_grav=-1.0, shrink=1, precision=0, n_initial=1, solver=1, box_align=1)
    sim = make_sim(cfg, 1)
    gen = torch.Generator(device="cuda:0").manual_seed(ng)
    old = torch.randn((ng,) * 3, generator=gen, dtype=torch.float64, device="cuda:0")
    f = torch.randn((ng,) * 3, generator=gen, dtype=torch.float64, device="cuda:0")
    sim.bind([[0.5 * box] * 3], [[0.0] * 3], [0])
    sim.shrink_radius((cells - 5) // 2 * h)
    st = sim.state()
    lo, hi = st["lo"], st["hi"]
    assert st["periodic"] == 0 and all(b - a + 1 == cells for a, b in zip(lo, hi))
    sim.phi.copy_(old)
    sim.rhs.copy_(f)
    sim.ade_sweep(lam, forward)
    new, old, f = sim.phi_numpy(), old.cpu().numpy(), f.cpu().numpy()
    inside = np.zeros(old.shape, dtype=bool)
    inside[lo[2]:hi[2] + 1, lo[1]:hi[1] + 1, lo[0]:hi[0] + 1] = True
    assert np.array_equal(new[~inside], old[~inside])
    scale = (1.0 + 3.0 * lam) * np.abs(new).max()
    # the bound of the periodic sweep's own test: 64 roundings of the terms
    assert _box_residual(old, new, f, lam, lo, hi, forward) <= 1e-14 * 64 * scale
    sim.close()


# Sweeps of several contexts at a time, each on a stream and thread of its own:
# their workgroups, which wait for one another within a sweep, share the compute
# units in any order.  Every sweep gives what it gives alone.
@pytest.mark.parametrize("ng,contexts,sweeps", [(128, 8, 12), (256, 6, 8), (512, 4, 3)])
def test_concurrent_sweeps(ng, contexts, sweeps):
    import threading

    import torch

    lam = 8.8
    cfg = lib_config(ng, 100.0, c_grav=-1.0, precision=0, n_initial=1, solver=1)
    gen = torch.Generator(device="cuda:0").manual_seed(ng)
    old = torch.randn((ng,) * 3, generator=gen, dtype=torch.float64, device="cuda:0")
    f = torch.randn((ng,) * 3, generator=gen, dtype=torch.float64, device="cuda:0")
    sims = []
    for _ in range(contexts):
        with torch.cuda.stream(torch.cuda.Stream()):
            sims.append(make_sim(cfg, 1))
    for sim in sims:
        sim.bind([[50.0, 50.0, 50.0]], [[0.0, 0.0, 0.0]], [0])
        sim.phi.copy_(old)
        sim.rhs.copy_(f)
    torch.cuda.synchronize()

    def run(sim):
        for q in range(sweeps):
            sim.ade_sweep(lam, q % 2 == 0)

    threads = [threading.Thread(target=run, args=(sim,)) for sim in sims[1:]]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    run(sims[0])                                 # alone
    torch.cuda.synchronize()
    assert not torch.equal(sims[0].phi, old)
    for sim in sims[1:]:
        assert torch.equal(sim.phi, sims[0].phi)
    for sim in sims:
        sim.close()


def _by_diagonals(u, f, lam, dtype):
    """The forward sweep of a periodic mesh in the given precision: diagonals of
    rows in order, cells of a row in order, c + a u of the cell before."""
    u, f, lam = u.astype(dtype), f.astype(dtype), dtype(lam)
    n = u.shape[0]
    co, inv = 1 - 3 * lam, 1 / (1 + 3 * lam)
    a = lam * inv
    for d in range(2 * n - 1):
        k = np.arange(max(0, d - n + 1), min(n - 1, d) + 1)
        j = d - k
        for i in range(n):
            s = (u[k, j, (i + 1) % n] + u[k, j - 1, i] + u[k, (j + 1) % n, i] + u[k - 1, j, i] +
                 u[(k + 1) % n, j, i])
            u[k, j, i] = (co * u[k, j, i] + lam * (s - f[k, j, i])) * inv + a * u[k, j, i - 1]
    return u


@pytest.mark.parametrize("lam", [0.05, 8.8, 1e3])
def test_rounding_of_a_smooth_field(lam):
    """A smooth field passes through many cells of a sweep with lam >> 1, and
    with it what the rounded coefficients add up to: the error is that of the
    update as written.  Its random part differs from order to order; a fifth
    covers it, where a coefficient rounded on its own added a third."""
    import torch

    ng = 64
    t = 2.0 * np.pi * np.arange(ng) / ng
    old = np.sin(t)[:, None, None] + np.cos(2 * t)[None, :, None] * np.sin(3 * t)[None, None, :]
    f = 0.01 * np.roll(old, 3, 1)
    cfg = lib_config(ng, 100.0, c_grav=-1.0, precision=0, n_initial=1, solver=1)
    sim = make_sim(cfg, 1)
    sim.bind([[50.0, 50.0, 50.0]], [[0.0, 0.0, 0.0]], [0], phi=old)
    sim.rhs.copy_(torch.as_tensor(f))
    sim.ade_sweep(lam, True)
    ref = _by_diagonals(old, f, lam, np.longdouble)
    plain = _by_diagonals(old, f, lam, np.float64)
    err, allowed = (float(np.sqrt(((v - ref) ** 2).mean())) for v in (sim.phi_numpy(), plain))
    assert err <= 1.2 * allowed
    sim.close()
