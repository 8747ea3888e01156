"""The FP64 force interpolation on its two load paths: waves whose particles'
rows lie inside the mesh (pairs of values) and waves with rows that wrap around
(single values), CIC and TSC, on a potential with a large constant part."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import pm

from helpers import lib_config, make_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("assignment", [0, 1])
@pytest.mark.parametrize("where", ["inside", "edges", "mixed"])
def test_force_against_oracle(assignment, where):
    import torch

    ng, box, n = 32, 100.0, 1000
    h = box / ng
    rng = np.random.default_rng(assignment + 10 * len(where))
    x = rng.uniform(4 * h, (ng - 4) * h, size=(n, 3))
    if where != "inside":
        rows = np.arange(n) if where == "edges" else np.arange(0, n, 200)
        x[rows, 0] = np.where(rng.random(len(rows)) < 0.5, rng.uniform(0, 1.5 * h, len(rows)),
                              rng.uniform(box - 1.5 * h, box, len(rows)))
    cfg = lib_config(ng, box, precision=1, n_initial=n, assignment=assignment)
    sim = make_sim(cfg, n)
    sim.bind(x, np.zeros((n, 3)), np.arange(n))
    phi = 1000.0 + rng.normal(size=(ng, ng, ng))
    sim.phi.copy_(torch.as_tensor(phi))
    got = sim.interp_force().cpu().numpy().T
    ref = pm.interpolate(x, pm.force_mesh(phi, h), ng, box, 14, True, "tsc" if assignment else "cic")
    # both sum differences of the same potential values; those have one
    # rounding each at most, and no sum has more than 81 terms
    u = 2.0 ** -53
    scale = np.abs(phi - 1000.0).max() / h
    assert np.abs(got - ref).max() <= 2 * 81 * 4 * u * scale
    sim.close()


@pytest.mark.parametrize("assignment", [0, 1])
def test_force_of_an_uneven_potential(assignment):
    """Potential values nine orders of magnitude apart, particles on nodes among
    them: each node's difference counts with its own rounding, not with that of
    the largest value around."""
    import torch

    ng, box, n = 32, 100.0, 20000
    h = box / ng
    rng = np.random.default_rng(7 + assignment)
    x = rng.uniform(0.0, box, size=(n, 3))
    x[:500] = np.floor(x[:500] / h) * h
    cfg = lib_config(ng, box, precision=1, n_initial=n, assignment=assignment)
    sim = make_sim(cfg, n)
    sim.bind(x, np.zeros((n, 3)), np.arange(n))
    phi = rng.normal(size=(ng,) * 3) * 10.0 ** rng.uniform(-6.0, 3.0, size=(ng,) * 3)
    sim.phi.copy_(torch.as_tensor(phi))
    got = sim.interp_force().cpu().numpy().T
    g = pm.force_mesh(phi, h)
    kind = "tsc" if assignment else "cic"
    ref = pm.interpolate(x, g, ng, box, cfg.frac_bits, True, kind)
    # a node's term has four roundings, and it passes through at most one sum
    # per node; on both sides
    nodes = 27 if assignment else 8
    bound = 2 * (nodes + 4) * 2.0**-53 * pm.interpolate(x, np.abs(g), ng, box, cfg.frac_bits, True, kind)
    assert np.all(np.abs(got - ref) <= bound)
    sim.close()
