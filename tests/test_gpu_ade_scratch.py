"""A multigrid solve on a frozen-exterior box after an ADE sweep of the same
context: the sweep's rows pass between workgroups through the workspace's
residual array, all over the mesh, and leave any bits there.  The solve gives
what it gives without the sweep, and so does what it records."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from synth import clustered_particles

from helpers import lib_config, make_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ng,radius", [(32, 9.3), (64, 23.6), (128, 41.3), (256, 90.2)])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("pre", [2, 3])
def test_solve_after_sweep(ng, radius, prec, pre):
    box, n, kappa = 10.0 * ng, 3000, 0.1
    x, p, ids = clustered_particles(n, box, 3, ng=ng, width_cells=1.0, lo=0.36 * box, hi=0.64 * box)
    cfg = lib_config(ng, box, c_grav=-1.0, shrink=1, precision=prec, n_initial=n, pre=pre)
    got = []
    for sweep in (False, True):
        sim = make_sim(cfg, n)
        sim.bind(x, p, ids)
        sim.shrink_radius(radius * box / ng)
        assert sim.state()["periodic"] == 0
        gen = torch.Generator(device="cuda:0").manual_seed(ng)
        phi0 = torch.randn((ng,) * 3, generator=gen, dtype=torch.float64, device="cuda:0")
        if sweep:
            # negative zeros and infinities among the values whose halves pass
            sim.phi.copy_(phi0)
            sim.rhs.copy_(phi0)
            sim.phi[::3, ::2, ::5] = -0.0
            sim.phi[ng // 2, ng // 2, ng // 2] = float("inf")
            sim.ade_sweep(8.8, True)
        sim.phi.copy_(phi0)
        sim.deposit()
        rec = torch.zeros(3 * ng**3, dtype=torch.float32, device="cuda:0")
        sim.record(rec, 1)
        st = sim.solve(kappa, 1.0)
        got.append((st["vcycles"], sim.phi.clone(), rec))
        sim.close()
    assert got[0][0] == got[1][0]
    assert torch.equal(got[0][1], got[1][1])
    assert torch.equal(got[0][2], got[1][2]) and bool(torch.isfinite(got[0][2]).all())
