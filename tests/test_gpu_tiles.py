"""Solves on the meshes whose every level runs in one launch down and one up:
the smallest mesh, one and several tiles a side, cycles that start from zero
(one per correction) and from the correction of the cycle before (four), boxes
whose faces cut the tiles, and a coarsest level solved by sweeps over tiles.
A pass that is wrong near a tile's faces costs cycles or does not converge."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import pm
from synth import clustered_particles, uniform_particles

from helpers import cond_periodic, lib_config, make_sim, rel_rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ng,kappa", [(8, 0.05), (16, 0.05), (32, 0.0), (64, 0.0), (64, 0.3)])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("per_outer", [1, 4])
def test_periodic(ng, kappa, prec, per_outer):
    box, tol = 100.0, 1e-8
    n = ng**3 // 2 + 5
    x, p, ids = uniform_particles(n, box, ng)
    cfg = lib_config(ng, box, precision=prec, tol=tol, n_initial=n, cycles_per_outer=per_outer)
    sim = make_sim(cfg, n)
    phi0 = np.random.default_rng(ng).normal(size=(ng,) * 3) * 1e-3
    sim.bind(x, p, ids, phi=phi0)
    sim.deposit()
    st = sim.solve(kappa, 1.0)
    ref = pm.solve_periodic(sim.rhs.cpu().numpy(), kappa)
    assert st["res"][0] <= tol
    assert rel_rms(sim.phi_numpy(), ref) <= cond_periodic(ng, kappa) * tol
    # V(2,2) cuts the residual at least fivefold per cycle: 12 for 1e-8
    assert st["vcycles"] <= 12
    sim.close()


@pytest.mark.parametrize("ng,radius", [(32, 9.3), (64, 20.1), (64, 23.6)])
@pytest.mark.parametrize("kappa", [0.02, 0.6])
@pytest.mark.parametrize("prec", [0, 1])
def test_box(ng, radius, kappa, prec):
    import torch

    box, tol, n = 10.0 * ng, 1e-8, 3000
    x, p, ids = clustered_particles(n, box, 3, ng=ng, width_cells=1.0, lo=0.36 * box, hi=0.64 * box)
    cfg = lib_config(ng, box, c_grav=-1.0, shrink=1, precision=prec, tol=tol, n_initial=n)
    sim = make_sim(cfg, n)
    phi0 = np.random.default_rng(ng).normal(size=(ng,) * 3) * 1e-2
    sim.bind(x, p, ids)
    sim.shrink_radius(radius * box / ng)
    st = sim.state()
    assert st["periodic"] == 0
    lo, hi = st["lo"], st["hi"]
    sim.phi.copy_(torch.as_tensor(phi0))
    sim.deposit()
    st = sim.solve(kappa, 1.0)
    sl = tuple(slice(lo[d], hi[d] + 1) for d in (2, 1, 0))
    rhs = np.zeros((ng,) * 3)
    rhs[sl] = sim.rhs.cpu().numpy()[sl]
    ref = pm.solve_box(phi0, rhs, lo, hi, kappa)
    got = sim.phi_numpy()
    out = np.ones(got.shape, dtype=bool)
    out[sl] = False
    assert np.array_equal(got[out], phi0[out])
    assert st["res"][0] <= tol and st["vcycles"] <= 14
    # ||phi - ref|| <= ||residual|| / smallest eigenvalue
    ext = max(b - a + 1 for a, b in zip(lo, hi))
    lam = kappa + 3 * (2 - 2 * np.cos(np.pi / (ext + 1)))
    err = np.linalg.norm(got[sl] - ref[sl])
    assert err <= 1.01 * tol * np.linalg.norm(rhs[sl]) / lam + 1e-12 * np.linalg.norm(ref[sl])
    sim.close()
