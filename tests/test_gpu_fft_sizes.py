"""The FFT solve at the mesh sizes where its transforms change form: 8 (rows as
complex lines), 16 and 32 (one and two radix stages a row), 1024 (three
exchanges a line), against torch's FP64 transforms of the same equation.

Tolerance: as for the other sizes, 1e-11 relative RMS (two exact FP64 solves)."""
from __future__ import annotations

import math

import pytest

from helpers import lib_config, make_sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ng", [8, 16, 32, 64, 1024])
def test_solve_against_torch(ng):
    import torch

    import paper_1709_04703_amd as P

    kappa = 0.2
    cfg = lib_config(ng, 100.0, precision=0, n_initial=1, solver=P.SDPM_SOLVER_FFT)
    sim = make_sim(cfg, 1)
    sim.bind([[50.0, 50.0, 50.0]], [[0.0, 0.0, 0.0]], [0])
    gen = torch.Generator(device="cuda:0").manual_seed(ng)
    phi0 = torch.randn((ng,) * 3, generator=gen, dtype=torch.float64, device="cuda:0")
    sim.phi.copy_(phi0)
    sim.counts.zero_()
    sim.solve(kappa, 0.0)                       # rhs = -kappa phi0
    assert torch.equal(sim.rhs, -kappa * phi0)
    s = 2.0 - 2.0 * torch.cos(2.0 * math.pi * torch.arange(ng, dtype=torch.float64, device="cuda:0") / ng)
    f = torch.fft.rfftn(phi0.mul_(-kappa))
    for k in range(ng):                         # plane by plane: 1024^3 of symbols is not needed at once
        f[k] /= -(s[k] + s[:, None] + s[None, :ng // 2 + 1]) - kappa
    ref = torch.fft.irfftn(f, s=(ng,) * 3)
    err = float((sim.phi - ref).norm() / ref.norm())
    assert err <= 1e-11
    sim.close()
    del sim, phi0, f, ref
    torch.cuda.empty_cache()


@pytest.mark.parametrize("ng", [8, 512])
def test_poisson_zero_mode(ng):
    """kappa = 0: the mean of the potential is zero and its Laplacian is the
    source without its mean."""
    import torch

    import paper_1709_04703_amd as P

    n = 4000
    cfg = lib_config(ng, 100.0, precision=1, n_initial=n, solver=P.SDPM_SOLVER_FFT)
    sim = make_sim(cfg, n)
    gen = torch.Generator(device="cuda:0").manual_seed(ng)
    x = torch.rand((n, 3), generator=gen, dtype=torch.float64, device="cuda:0") * 100.0
    sim.bind(x.cpu().numpy(), torch.zeros((n, 3)).numpy(), list(range(n)))
    sim.deposit()
    sim.solve(0.0, 1.0)
    phi, rhs = sim.phi, sim.rhs
    lap = sum(torch.roll(phi, s, d) for d in range(3) for s in (1, -1)) - 6.0 * phi
    r = rhs - rhs.mean() - lap
    assert float(r.norm() / rhs.norm()) <= 1e-11
    assert abs(float(phi.mean())) <= 1e-12 * float(phi.abs().max())
    sim.close()


def test_errors_of_other_callers():
    """An error that another library left in the thread (refused on the host: a
    device that does not exist) is not the FFT solver's: contexts are made and
    solves run as without it."""
    import ctypes

    import numpy as np
    import torch

    import paper_1709_04703_amd as P

    ng, kappa = 16, 0.2
    cfg = lib_config(ng, 100.0, precision=0, n_initial=1, solver=P.SDPM_SOLVER_FFT)
    sim = make_sim(cfg, 1)
    phi0 = np.random.default_rng(1).normal(size=(ng,) * 3)
    sim.bind([[50.0, 50.0, 50.0]], [[0.0, 0.0, 0.0]], [0], phi=phi0)
    sim.counts.zero_()
    other = torch.empty_like(sim.workspace)
    torch.cuda.synchronize()
    lib = P.library()                           # its symbols include the runtime's
    ctx = ctypes.c_void_p()
    try:
        assert lib.hipSetDevice(1 << 20) != 0
        sim.solve(kappa, 0.0)
        assert lib.hipSetDevice(1 << 20) != 0
        assert lib.sdpm_create(ctypes.byref(cfg), ctypes.c_void_p(other.data_ptr()), sim.ws_bytes,
                               ctypes.c_void_p(sim.stream.cuda_stream), ctypes.byref(ctx)) == 0
    finally:
        lib.hipGetLastError()
    assert lib.sdpm_destroy(ctx) == 0
    phi = sim.phi_numpy()
    lap = sum(np.roll(phi, s, d) for d in range(3) for s in (1, -1)) - 6.0 * phi
    assert np.abs(lap - kappa * phi + kappa * phi0).max() <= 1e-13 * np.abs(phi0).max()
    sim.close()
