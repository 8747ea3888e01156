"""Solves on a mesh whose finest levels take the fused four-sweep passes, the
last with the coarser level's correction prolonged in it: periodic, and
frozen-exterior boxes whose faces lie inside a column's units and rows and on
planes of either parity, from zero and from the correction of the cycle before.  The result
is checked by its residual, evaluated in NumPy, and every V(2,2) cycle has to
cut the residual as the separate sweeps do."""
from __future__ import annotations

import numpy as np
import pytest

from synth import clustered_particles

from helpers import lib_config, make_sim

pytestmark = pytest.mark.gpu


def _relative_residual(phi, rhs, kappa, sl):
    lap = sum(np.roll(phi, s, ax) for ax in range(3) for s in (1, -1)) - 6.0 * phi
    r = (rhs - (lap - kappa * phi))[sl]
    return np.linalg.norm(r) / np.linalg.norm(rhs[sl])


@pytest.mark.parametrize("radius", [None, 64.6, 65.5, 90.2])
@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("kappa", [0.0, 0.09])
@pytest.mark.parametrize("per_outer", [1, 3])
def test_solve_256(radius, prec, kappa, per_outer):
    import torch

    ng, box, n, tol = 256, 2560.0, 40000, 1e-9
    x, p, ids = clustered_particles(n, box, 9, ng=ng, width_cells=2.0, lo=0.36 * box, hi=0.64 * box)
    # (kappa = 0 on boxes that the coarser meshes cannot hold does not converge,
    # whatever kernel sweeps them: aligned boxes there)
    align = dict(box_align=1) if kappa else {}
    cfg = lib_config(ng, box, precision=prec, tol=tol, n_initial=n, shrink=0 if radius is None else 1,
                     cycles_per_outer=per_outer, **align)
    sim = make_sim(cfg, n)
    sim.bind(x, p, ids)
    if radius is not None:
        sim.shrink_radius(radius * box / ng)
    st = sim.state()
    assert st["periodic"] == (radius is None)
    lo, hi = st["lo"], st["hi"]
    phi0 = np.random.default_rng(3).normal(size=(ng,) * 3) * 1e-2
    sim.phi.copy_(torch.as_tensor(phi0))
    sim.deposit()
    st = sim.solve(kappa, 1.0)
    sl = tuple(slice(lo[d], hi[d] + 1) for d in (2, 1, 0))
    phi, rhs = sim.phi_numpy(), sim.rhs.cpu().numpy()
    true = _relative_residual(phi, rhs, kappa, sl)
    assert true <= tol * (1 + 1e-6)
    assert abs(st["res"][0] - true) <= max(0.05 * tol, 1e-3 * true)
    # a cycle cuts the residual at least sevenfold; the start's is below 1e3
    assert st["vcycles"] <= int(np.ceil(np.log(1e3 / tol) / np.log(7.0)))
    out = np.ones(phi.shape, dtype=bool)
    out[sl] = False
    assert np.array_equal(phi[out], phi0[out])
    sim.close()
