"""The work that a user of the library has it do, as cases that can be timed and compared.

Kinds of case:
  run        a whole small simulation: bind host arrays, initial potential, all steps
  step       one step of a running simulation on the periodic mesh (any solver, scheme, precision)
  shrink     one step in the shrinking phase: frozen-exterior box, removal, lightcone output
  solve      one multigrid solve from a zero guess (the initial potential, a field update)
  ade        a forward and a backward sweep of the paper's explicit gravity integrator
  particles  re-sort, mass deposit and force interpolation of a particle set of any size
  pk         the power spectrum of a particle set
  train      one training step of the warm-start net on one recorded pair
  conv       one layer of that net, forward and data gradient

Inputs are drawn on the GPU from the case's seed: Zel'dovich positions and momenta of a
Lambda-CDM-like spectrum for the simulations, smooth fields and blobs for the single calls.
exact() evaluates the same formulas with plain torch and numpy in 64 bits.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_1709_04703_amd import _lib as L

DEV = "cuda:0"
OM, OL, HUBBLE = 0.3, 0.7, 0.7
C_LIGHT = 2997.92458
FRAC_BITS = 14
F64 = torch.float64


# ------------------------------------------------------------------ the cases
def listed():
    """The range a user covers, smallest to largest."""
    step = dict(kind="step", box=2000.0, a0=0.02, steps=1000, c_grav=-1.0, fp64=False, tsc=False,
                solver="mg", extrap=True, sort_every=20)
    return [
        # the smallest simulation: 32^3 particles, 100 Mpc/h, FP64, static gravity, all of its
        # 20 steps, arrays from the host as a program has them (latency and launches count)
        dict(name="run_32_fp64", kind="run", ng=32, n1d=32, box=100.0, a0=0.02, steps=20,
             c_grav=0.0, fp64=True, tol=1e-10),
        # a step of the ordinary 128^3 run, a particle lattice that is not the mesh's
        dict(step, name="step_128", ng=128, n1d=125),
        # 256^3: the standard FFT solver, and the careful settings (FP64 throughout, TSC)
        dict(step, name="step_256_fft", ng=256, n1d=256, solver="fft", extrap=False),
        dict(step, name="step_256_fp64_tsc", ng=256, n1d=251, fp64=True, tsc=True, extrap=False),
        # the benchmark's workload: 512^3 particles on a 512^3 mesh, 200 steps from z = 49
        dict(step, name="step_512", ng=512, n1d=512, steps=200),
        # the same run's late phase: most particles are gone, the box shrinks, records are written
        dict(name="shrink_512", kind="shrink", ng=512, n1d=512, box=2000.0, a0=0.8, steps=1000,
             c_grav=-1.0, sort_every=20),
        # an initial potential: Poisson's equation from a zero guess
        dict(name="solve_256", kind="solve", ng=256, n=2000003, kappa_h2=0.0, fp64=False),
        # the paper's own integrator
        dict(name="ade_256", kind="ade", ng=256, lam=8.8),
        # the particle calls on a clustered set of any size
        dict(name="particles_256", kind="particles", ng=256, n=5000011, tsc=False, fp64=False),
        # a snapshot's power spectrum with both corrections
        dict(name="pk_256", kind="pk", ng=256, n=4000037, shot=True, jing=True),
        # the warm-start net: training on 128^3 pairs, one layer at 128^3 both ways
        dict(name="train_128", kind="train", ng=128),
        dict(name="conv_128", kind="conv", ng=128, gain=1.0),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["run", "step", "step", "step", "shrink", "solve", "ade", "particles",
                       "particles", "pk", "train", "conv"])
    if kind == "run":
        ng = rng.choice([16, 32, 64])
        return dict(kind=kind, ng=ng, n1d=rng.randint(9, ng), box=rng.uniform(100.0, 500.0),
                    a0=rng.choice([0.02, 0.05]), steps=rng.randint(8, 20),
                    c_grav=rng.choice([0.0, -1.0]), fp64=rng.random() < 0.5, tol=1e-10)
    if kind == "step":
        ng = rng.choice([64, 128, 128, 256, 256, 512])
        solver = rng.choice(["mg", "mg", "mg", "fft", "ade"])
        return dict(kind=kind, ng=ng, n1d=rng.randint(ng // 2, ng), box=rng.uniform(500.0, 4000.0),
                    a0=rng.uniform(0.02, 0.2), steps=rng.choice([200, 500, 1000]), c_grav=-1.0,
                    fp64=rng.random() < 0.3, tsc=rng.random() < 0.3, solver=solver,
                    extrap=solver == "mg" and rng.random() < 0.6,
                    sort_every=rng.choice([0, 10, 20, 20]))
    if kind == "shrink":
        ng = rng.choice([128, 256, 512])
        return dict(kind=kind, ng=ng, n1d=rng.randint(ng // 2, ng), box=2000.0,
                    a0=rng.uniform(0.72, 0.85), steps=rng.choice([500, 1000]), c_grav=-1.0,
                    sort_every=20)
    if kind == "solve":
        return dict(kind=kind, ng=rng.choice([32, 64, 128, 256, 512]), n=logint(20000, 5000000),
                    kappa_h2=rng.choice([0.0, math.exp(rng.uniform(math.log(1e-2), math.log(1.0)))]),
                    fp64=rng.random() < 0.4)
    if kind == "ade":
        return dict(kind=kind, ng=rng.choice([32, 64, 128, 256]),
                    lam=math.exp(rng.uniform(math.log(0.3), math.log(100.0))))
    if kind == "particles":
        return dict(kind=kind, ng=rng.choice([64, 128, 256, 512]), n=logint(20000, 20000000),
                    tsc=rng.random() < 0.4, fp64=rng.random() < 0.4)
    if kind == "pk":
        return dict(kind=kind, ng=rng.choice([64, 128, 256]), n=logint(50000, 10000000),
                    shot=rng.random() < 0.7, jing=rng.random() < 0.7)
    if kind == "train":
        return dict(kind=kind, ng=rng.choice([32, 64, 128]), lr=math.exp(rng.uniform(-9.0, -6.0)))
    return dict(kind=kind, ng=rng.choice([32, 64, 128, 256]), gain=rng.uniform(0.5, 2.0))


def work(case):
    """Bytes and operations of one pass that no implementation can do without."""
    k, ng = case["kind"], case["ng"]
    v = float(ng) ** 3
    pb = 8 if case.get("fp64") else 4
    nodes = 27 if case.get("tsc") else 8
    if k in ("run", "step", "shrink"):
        n, cells = float(case["n1d"]) ** 3, v
        if k == "shrink":    # the sphere's share of particles and of cells
            r = _lightcone_radius(case["a0"])
            f = min(1.0, 4.0 / 3.0 * math.pi * r ** 3 / case["box"] ** 3)
            n, cells = n * f, v * min(1.0, (2.0 * r / case["box"]) ** 3)
        # positions and momenta in and out; potential in and out, density and source out
        b = n * 2 * (24 + 3 * pb) + cells * (16 + 16)
        f = n * nodes * 12 + cells * 60
        s = case["steps"] if k == "run" else 1
        return {"bytes": float(b * s), "flops": float(f * s)}
    if k == "solve":
        return {"bytes": v * 24, "flops": v * 60}
    if k == "ade":
        return {"bytes": v * 48, "flops": v * 24}
    if k == "particles":
        n = float(case["n"])
        # sort: every array in and out; deposit: positions; force: positions in, force out
        return {"bytes": n * (2 * (24 + 3 * pb + 4) + 24 + 48) + v * 16, "flops": n * nodes * 16}
    if k == "pk":
        return {"bytes": float(case["n"]) * 24 + v * 24, "flops": v * 2.5 * math.log2(v)}
    layer = 2.0 * 27 * 16 * 16 * v
    if k == "train":
        # 5 layers forward, 4 data gradients, 5 weight gradients; the method's channels only
        fwd = 2.0 * 27 * (3 * 16 + 3 * 256 + 16) * v
        return {"bytes": v * (12 + 14 * 32), "flops": 3.0 * fwd}
    return {"bytes": v * 32 * 5, "flops": 2.0 * layer}


# ----------------------------------------------------------------- cosmology
def _e(a):
    return np.sqrt(OM / a ** 3 + (1.0 - OM - OL) / a ** 2 + OL)


_GLX, _GLW = np.polynomial.legendre.leggauss(64)


def _dtau(a0, a1):
    """Conformal time between two scale factors, in u = sqrt(a)."""
    edges = np.linspace(math.sqrt(a0), math.sqrt(a1), 9)
    tot = 0.0
    for lo, hi in zip(edges[:-1], edges[1:]):
        u = 0.5 * (lo + hi) + 0.5 * (hi - lo) * _GLX
        a = u * u
        tot += float(np.sum(_GLW * 2.0 * u / (a * a * _e(a)))) * 0.5 * (hi - lo)
    return tot


def _lightcone_radius(a):
    return 0.0 if a >= 1.0 else C_LIGHT * _dtau(a, 1.0)


def _scalars(c, a, da):
    a1, h = a + da, c["box"] / c["ng"]
    dtau = _dtau(a, a1)
    lo, hi = a, a1
    mid = 0.5 * (lo + hi)
    for _ in range(60):
        step = (_dtau(a, mid) - 0.5 * dtau) * mid * mid * float(_e(mid))
        mid -= step
        if abs(step) <= 4e-16 * mid:
            break
    k1 = k2 = 0.0
    if c["c_grav"] != 0.0:
        cg = 0.019 * h * C_LIGHT if c["c_grav"] < 0.0 else c["c_grav"]
        den = cg * cg * 0.5 * dtau
        k1 = 3.0 * mid * float(_e(mid)) * h * h / den
        k2 = 3.0 * a1 * float(_e(a1)) * h * h / den
    return dtau, mid, 1.5 * OM / mid, k1, k2


def _growth(a):
    """(D, f): growing mode with D(1) = 1, from its integral."""
    def g(b):
        x = (np.arange(20000) + 0.5) / 20000 * b
        return float(_e(b)) * float(np.sum((x * _e(x)) ** -3.0)) * b / 20000
    eps = 1e-4
    f = (math.log(g(a * (1 + eps))) - math.log(g(a * (1 - eps)))) / (2 * eps)
    return g(a) / g(1.0), f


def _shape(k, lib):
    """Zero-baryon Eisenstein & Hu (1998) k T(k)^2 for an array library."""
    q = k * (2.7255 / 2.7) ** 2 / (OM * HUBBLE)
    l0 = lib.log(2.0 * math.e + 1.8 * q)
    t = l0 / (l0 + (14.2 + 731.0 / (1.0 + 62.5 * q)) * q * q)
    return k * t * t


def _amplitude():
    k = np.exp(np.linspace(math.log(1e-5), math.log(1e2), 20001))
    x = 8.0 * k
    w = np.where(x < 1e-3, 1.0, 3.0 * (np.sin(x) - x * np.cos(x)) / np.maximum(x, 1e-12) ** 3)
    y = k ** 3 * _shape(k, np) * w * w / (2.0 * math.pi ** 2)
    s2 = float(np.sum(0.5 * (y[1:] + y[:-1]))) * math.log(k[1] / k[0])
    return 0.8 ** 2 / s2


def _particles(n1d, box, a, seed, fp64):
    """Zel'dovich positions (3, n) in [0, box) and momenta (3, n) on an n1d^3 lattice."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    w = torch.randn((n1d,) * 3, generator=gen, device=DEV, dtype=F64)
    wk = torch.fft.rfftn(w)
    del w
    kf = 2.0 * math.pi / box
    k1 = torch.fft.fftfreq(n1d, 1.0 / n1d, device=DEV, dtype=F64) * kf
    kx = (torch.fft.rfftfreq(n1d, 1.0 / n1d, device=DEV, dtype=F64) * kf)[None, None, :]
    ky, kz = k1[None, :, None], k1[:, None, None]
    kk = torch.sqrt(kx * kx + ky * ky + kz * kz)
    kk[0, 0, 0] = 1.0
    wk *= torch.sqrt(_amplitude() * _shape(kk, torch) / (box / n1d) ** 3) / (kk * kk)
    wk[0, 0, 0] = 0.0
    if n1d % 2 == 0:
        m = n1d // 2
        wk[m], wk[:, m], wk[:, :, m] = 0.0, 0.0, 0.0
    del kk
    d, f = _growth(a)
    vel = a * a * float(_e(a)) * f
    n = n1d ** 3
    x = torch.empty((3, n), dtype=F64, device=DEV)
    p = torch.empty((3, n), dtype=F64 if fp64 else torch.float32, device=DEV)
    q = (torch.arange(n1d, device=DEV, dtype=F64) + 0.5) * (box / n1d)
    for ax, k in enumerate((kx, ky, kz)):
        psi = torch.fft.irfftn(1j * k * wk, s=(n1d,) * 3) * d
        view = [1, 1, 1]
        view[2 - ax] = n1d
        pos = torch.remainder(psi + q.view(view), box)
        pos[pos >= box] = 0.0
        x[ax] = pos.reshape(-1)
        p[ax] = (psi * vel).reshape(-1).to(p.dtype)
        del psi, pos
    return x, p


def _blobs(n, box, seed):
    """Half of the particles uniform, half in Gaussian blobs, in [0, box)."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    x = torch.rand((3, n), generator=gen, device=DEV, dtype=F64) * box
    half, nb = n // 2, 200
    centre = torch.rand((3, nb), generator=gen, device=DEV, dtype=F64) * box
    which = torch.randint(0, nb, (half,), generator=gen, device=DEV)
    off = torch.randn((3, half), generator=gen, device=DEV, dtype=F64) * (0.01 * box)
    x[:, :half] = torch.remainder(centre[:, which] + off, box)
    x[x >= box] = 0.0
    return x


def _smooth(ng, seed, amp):
    """A smooth random periodic field of the given rms."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    f = torch.fft.rfftn(torch.randn((ng,) * 3, generator=gen, device=DEV, dtype=F64))
    k = torch.fft.fftfreq(ng, 1.0 / ng, device=DEV, dtype=F64)
    kx = torch.fft.rfftfreq(ng, 1.0 / ng, device=DEV, dtype=F64)
    k2 = kx[None, None, :] ** 2 + k[None, :, None] ** 2 + k[:, None, None] ** 2
    k2[0, 0, 0] = 1.0
    f = f / k2
    f[0, 0, 0] = 0.0
    v = torch.fft.irfftn(f, s=(ng,) * 3)
    return (v * (amp / v.std())).contiguous()


# --------------------------------------------------------------- simulations
class _State:
    pass


def _config(c, n):
    kw = dict(n_initial=n, c_grav=c.get("c_grav", 0.0), tol=c.get("tol", 1e-8),
              precision=L.SDPM_PLAIN_FP64 if c.get("fp64") else L.SDPM_MIXED,
              assignment=L.SDPM_ASSIGN_TSC if c.get("tsc") else L.SDPM_ASSIGN_CIC,
              sort_every=c.get("sort_every", 0), shrink=1 if c["kind"] == "shrink" else 0,
              solver={"mg": L.SDPM_SOLVER_IMPLICIT, "fft": L.SDPM_SOLVER_FFT,
                      "ade": L.SDPM_SOLVER_ADE}[c.get("solver", "mg")])
    if c.get("extrap") or c["kind"] == "shrink":
        kw["warm_start"] = L.SDPM_WS_EXTRAP
    return L.config_default(c["ng"], c.get("box", 100.0), **kw)


def _bind(sim, x, p):
    """Device arrays into the simulation's own buffers."""
    n = x.shape[1]
    sim.x[:, :n].copy_(x)
    if p is not None:
        sim.p[:, :n].copy_(p)
    else:
        sim.p.zero_()
    torch.arange(n, out=sim.ids[:n])
    parts = L.Particles()
    for d in range(3):
        parts.x[d], parts.p[d] = sim.x[d].data_ptr(), sim.p[d].data_ptr()
    parts.id, parts.capacity = sim.ids.data_ptr(), n
    fields = L.Fields(sim.phi.data_ptr(), sim.rhs.data_ptr(), sim.counts.data_ptr())
    L.check(sim.lib.sdpm_bind(sim.ctx, ctypes.byref(parts), ctypes.byref(fields), n), sim.ctx)
    sim.n_active = n


def _start(s):
    """(Re)starts a simulation at its first step."""
    s.sim.phi.zero_()
    _bind(s.sim, s.x0, s.p0)
    s.a = s.case["a0"]
    s.sim.init_potential(s.a)
    if s.case["kind"] == "shrink":
        m = s.lc["id"].numel()
        lc = L.Lightcone()
        lc.id, lc.a, lc.capacity = s.lc["id"].data_ptr(), s.lc["a"].data_ptr(), m
        for d in range(3):
            lc.x[d], lc.p[d] = s.lc["x"][d].data_ptr(), s.lc["p"][d].data_ptr()
        L.check(s.sim.lib.sdpm_set_lightcone(s.sim.ctx, ctypes.byref(lc)), s.sim.ctx)


def prepare(case, seed):
    k, ng = case["kind"], case["ng"]
    s = _State()
    s.case = case
    if k in ("run", "step", "shrink"):
        n = case["n1d"] ** 3
        s.x0, s.p0 = _particles(case["n1d"], case["box"], case["a0"], seed, case.get("fp64", False))
        s.sim = L.Simulation(_config(case, n), n, DEV)
        s.da = (1.0 - (0.02 if k == "shrink" else case["a0"])) / case["steps"]
        if k == "run":
            s.host = (np.ascontiguousarray(s.x0.T.cpu().numpy()),
                      np.ascontiguousarray(s.p0.T.double().cpu().numpy()),
                      np.arange(n, dtype=np.uint32))
            s.edges = np.linspace(case["a0"], 1.0, case["steps"] + 1)
        else:
            if k == "shrink":
                s.lc = dict(id=torch.zeros(n, dtype=torch.int32, device=DEV),
                            a=torch.zeros(n, dtype=F64, device=DEV),
                            x=torch.zeros((3, n), dtype=F64, device=DEV),
                            p=torch.zeros((3, n), dtype=F64, device=DEV))
            _start(s)
    elif k == "solve":
        n = case["n"]
        s.sim = L.Simulation(_config(case, n), n, DEV)
        _bind(s.sim, _blobs(n, 100.0, seed), None)
        s.sim.deposit()
    elif k == "ade":
        s.sim = L.Simulation(_config(case, 1), 1, DEV)
        _bind(s.sim, torch.full((3, 1), 50.0, dtype=F64, device=DEV), None)
        s.sim.phi.copy_(_smooth(ng, seed, 1.0))
        s.sim.rhs.copy_(_smooth(ng, seed + 7777, 0.01))
    elif k == "particles":
        n = case["n"]
        c = dict(case, sort_every=20)
        s.sim = L.Simulation(_config(c, n), n, DEV)
        _bind(s.sim, _blobs(n, 100.0, seed), torch.ones((3, n), device=DEV))
        s.sim.phi.copy_(_smooth(ng, seed, 1.0))
    elif k == "pk":
        s.x = _blobs(case["n"], 100.0, seed)
    else:
        gen = torch.Generator(device=DEV).manual_seed(int(seed))
        v = ng ** 3

        def rnd(*shape):
            return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32)

        s.w = rnd(5, 27 * 256 + 16) * math.sqrt(2.0 / (27 * 16))
        if k == "train":
            s.r = (_smooth(ng, seed, 1.0) + 0.3 * rnd(ng, ng, ng)).float().contiguous()
            s.phi = _smooth(ng, seed + 7777, 1.0).float().contiguous()
            s.target = (0.5 * _smooth(ng, seed + 5555, 1.0)).float().contiguous()
            w0 = s.w[0, :27 * 256].view(27, 16, 16)
            w0[:, 3:, :] = 0.0
            w0 *= math.sqrt(16 / 3)
            s.w[4, :27 * 256].view(27, 16, 16)[:, :, 1:] = 0.0
            s.w[4, 27 * 256 + 1:] = 0.0
            s.w[:, 27 * 256:] *= 0.1
            s.params = s.w.reshape(-1).contiguous()
            s.m1 = rnd(s.params.numel()) * 1e-3
            s.m2 = rnd(s.params.numel()) ** 2 * 1e-5 + 1e-6
            s.act0 = torch.zeros((v, 16), dtype=torch.int16, device=DEV)
            s.scratch = torch.zeros(L.net_scratch_bytes(ng), dtype=torch.uint8, device=DEV)
            s.loss = torch.zeros(1, dtype=torch.float32, device=DEV)
            s.step, s.lr = 5, case.get("lr", 1e-3)
        else:
            s.inp = torch.relu(rnd(v, 16)).bfloat16().view(torch.int16)
            s.grad = rnd(v, 16).bfloat16().view(torch.int16)
            s.weight = case["gain"] * s.w[0, :27 * 256]
            s.bias = s.w[0, 27 * 256:].contiguous()
            s.out = torch.empty((v, 16), dtype=torch.int16, device=DEV)
            s.back = torch.empty((v, 16), dtype=torch.int16, device=DEV)
    return s


def run(s):
    c = s.case
    k, ng = c["kind"], c["ng"]
    if k == "run":
        sim = s.sim
        sim.bind(*s.host)
        sim.init_potential(s.edges[0])
        for a, b in zip(s.edges[:-1], s.edges[1:]):
            sim.step(a, b - a)
        return [sim.x, sim.p, sim.phi]
    if k in ("step", "shrink"):
        if s.a + s.da > 1.0 + 1e-12:
            _start(s)         # the run is over: the next one begins
        s.sim.step(s.a, min(s.da, 1.0 - s.a))
        s.a += s.da
        out = [s.sim.x, s.sim.p, s.sim.phi, s.sim.ids]
        return out + [s.lc["a"], s.lc["x"], s.lc["p"], s.lc["id"]] if k == "shrink" else out
    if k == "solve":
        s.sim.phi.zero_()
        s.sim.solve(c["kappa_h2"], 1.0)
        return [s.sim.phi, s.sim.rhs]
    if k == "ade":
        s.sim.ade_sweep(c["lam"], True)
        s.sim.ade_sweep(c["lam"], False)
        return s.sim.phi
    if k == "particles":
        s.sim.sort()
        s.sim.deposit()
        g = s.sim.interp_force()
        return [s.sim.x, s.sim.p, s.sim.ids, s.sim.counts, g]
    if k == "pk":
        r = L.power_spectrum(s.x, 100.0, ng, c["shot"], c["jing"])
        return [r["k"], r["p"], r["p_raw"], r["modes"]]
    if k == "train":
        L.net_prep(ng, s.r, s.phi, 0.9, 1.1, 0.113, s.act0)
        L.net_train_step(ng, s.params, s.m1, s.m2, s.step, s.lr, s.act0, s.target, 0.8, s.scratch,
                         s.loss)
        s.step += 1
        return [s.params, s.m1, s.m2, s.loss]
    L.conv3d(ng, s.inp, s.weight, s.bias, L.CONV_RELU, None, s.out)
    L.conv3d(ng, s.grad, s.weight, None, L.CONV_BACKWARD_DATA | L.CONV_MASK, s.inp, s.back)
    return [s.out.view(torch.bfloat16), s.back.view(torch.bfloat16)]


# ------------------------------------------------------------- 64-bit values
def _axis(x, ng, box, tsc, periodic):
    """First node, fixed-point weights per node, along one axis."""
    one = 1 << FRAC_BITS
    u = torch.floor(x * (float(ng * one) / box)).long()
    if periodic:
        u = u & (ng * one - 1)
    if not tsc:
        q = u & (one - 1)
        return u >> FRAC_BITS, [one - q, q]
    node = (u + one // 2) >> FRAC_BITS
    d = u - (node << FRAC_BITS)
    wm = ((one // 2 - d) ** 2 + one) >> (FRAC_BITS + 1)
    wp = ((one // 2 + d) ** 2 + one) >> (FRAC_BITS + 1)
    return node - 1, [wm, one - wm - wp, wp]


def _nodes(x, lo, hi, ng, box, tsc, periodic):
    """(flat node index, weight) for each node of particles [lo, hi)."""
    ax = [_axis(x[d, lo:hi], ng, box, tsc, periodic) for d in range(3)]
    m = ng - 1
    for k, wz in enumerate(ax[2][1]):
        for j, wy in enumerate(ax[1][1]):
            row = (((ax[2][0] + k) & m) * ng + ((ax[1][0] + j) & m)) * ng
            wzy = wz * wy
            for i, wx in enumerate(ax[0][1]):
                yield row + ((ax[0][0] + i) & m), wzy * wx


_CHUNK = 1 << 24


def _deposit(x, n, ng, box, tsc, periodic=True):
    counts = torch.zeros(ng ** 3, dtype=torch.int64, device=DEV)
    for lo in range(0, n, _CHUNK):
        for idx, w in _nodes(x, lo, min(n, lo + _CHUNK), ng, box, tsc, periodic):
            counts.index_add_(0, idx, w)
    return counts.view(ng, ng, ng)


def _force(x, n, phi, ng, box, tsc, periodic=True):
    g = torch.zeros((3, n), dtype=F64, device=DEV)
    inv = ng / (2.0 * box)
    for d in range(3):
        f = ((torch.roll(phi, 1, 2 - d) - torch.roll(phi, -1, 2 - d)) * inv).reshape(-1)
        for lo in range(0, n, _CHUNK):
            hi = min(n, lo + _CHUNK)
            for idx, w in _nodes(x, lo, hi, ng, box, tsc, periodic):
                g[d, lo:hi] += w.double() * f[idx]
    return g * 2.0 ** (-3 * FRAC_BITS)


def _solve(rhs, kappa):
    """Periodic (Lap - kappa) phi = rhs."""
    ng = rhs.shape[0]
    lam = 2.0 - 2.0 * torch.cos(2.0 * math.pi * torch.arange(ng, device=DEV, dtype=F64) / ng)
    f = torch.fft.rfftn(rhs)
    sym = -(lam[:, None, None] + lam[None, :, None] + lam[None, None, :ng // 2 + 1]) - kappa
    if kappa == 0.0:
        sym[0, 0, 0] = 1.0
        f[0, 0, 0] = 0.0
    return torch.fft.irfftn(f / sym, s=(ng,) * 3)


def _dst(v, dim):
    n = v.shape[dim]
    shape = list(v.shape)
    shape[dim] = 1
    z = torch.zeros(shape, dtype=F64, device=DEV)
    f = torch.fft.rfft(torch.cat([z, v, z, -v.flip(dim)], dim), dim=dim)
    return -f.imag.narrow(dim, 1, n).contiguous()


def _solve_box(phi, rhs, lo, hi, kappa):
    """The same on the cells lo..hi (x, y, z) with the exterior values of phi frozen."""
    sl = tuple(slice(lo[d], hi[d] + 1) for d in (2, 1, 0))
    b = rhs[sl].clone()
    for d in range(3):
        ax = 2 - d
        for at, edge in ((lo[d] - 1, 0), (hi[d] + 1, b.shape[ax] - 1)):
            out = list(sl)
            out[ax] = at
            b.select(ax, edge).sub_(phi[tuple(out)])
    sym = -kappa
    for ax in range(3):
        n = b.shape[ax]
        view = [1, 1, 1]
        view[ax] = n
        lam = 2.0 - 2.0 * torch.cos(math.pi * torch.arange(1, n + 1, device=DEV, dtype=F64) / (n + 1))
        sym = sym - lam.view(view)
        b = _dst(b, ax)
    b = b / sym
    for ax in range(3):
        b = _dst(b, ax) / (2.0 * (b.shape[ax] + 1))
    out = phi.clone()
    out[sl] = b
    return out


def _spread(v):
    out = torch.zeros_like(v)
    for b in range(11):
        out |= ((v >> b) & 1) << (3 * b)
    return out


def _sorted_order(x, n, c):
    """The re-sort's order: Morton order of blocks, then cell rows, stable."""
    ng = c["ng"]
    sh = 4 if ng >= 64 else 0
    cell = [torch.floor(x[d, :n] * (ng / c["box"])).clamp_(0, ng - 1).long() for d in range(3)]
    key = _spread(cell[0] >> sh) | (_spread(cell[1] >> sh) << 1) | (_spread(cell[2] >> sh) << 2)
    m = (1 << sh) - 1
    key = (key << (2 * sh)) | ((cell[2] & m) << sh) | (cell[1] & m)
    return torch.sort(key.to(torch.int32), stable=True).indices


class _Exact:
    """A simulation in 64 bits."""

    def __init__(self, c, x, p):
        self.c, self.x, self.p = c, x.clone(), p.double()
        self.n = x.shape[1]
        self.n0 = self.n
        self.ids = torch.arange(self.n, dtype=torch.int32, device=DEV)
        self.phi = torch.zeros((c["ng"],) * 3, dtype=F64, device=DEV)
        self.box = None

    def source(self, counts, s, kappa):
        c = self.c
        h = c["box"] / c["ng"]
        scale = s * h * h / (self.n0 / c["ng"] ** 3 * 2.0 ** (3 * FRAC_BITS))
        off = s * h * h * (1.0 if self.box else self.n / self.n0)
        return counts.double() * scale - off - kappa * self.phi

    def solve(self, rhs, kappa):
        return _solve_box(self.phi, rhs, *self.box, kappa) if self.box else _solve(rhs, kappa)

    def permute(self, order, n):
        self.x[:, :n] = self.x[:, :n][:, order]
        self.p[:, :n] = self.p[:, :n][:, order]
        self.ids[:n] = self.ids[:n][order]

    def shrink(self, r):
        """Particles outside the sphere go last, in order; returns how many."""
        c, n = self.c, self.n
        o = 0.5 * c["box"]
        d2 = ((self.x[0, :n] - o) ** 2 + (self.x[1, :n] - o) ** 2) + (self.x[2, :n] - o) ** 2
        keep = d2 <= r * r
        self.permute(torch.cat([keep.nonzero()[:, 0], (~keep).nonzero()[:, 0]]), n)
        self.n = int(keep.sum())
        h = c["box"] / c["ng"]
        lv = max(2, min(int(math.log2(c["ng"])) - 3, 12))
        al = 1 << (lv - 1)
        lo = math.floor((o - r) / h) - 2 - 1
        hi = math.floor((o + r) / h) + 2 + 1
        lo, hi = lo // al * al + 1, -(-hi // al) * al - 1
        if lo >= 1 and hi <= c["ng"] - 2:
            if self.box:
                lo, hi = max(lo, self.box[0][0]), min(hi, self.box[1][0])
            self.box = ([lo] * 3, [hi] * 3)
        return n - self.n

    def start(self, a):
        c = self.c
        if c["kind"] == "shrink":
            self.shrink(_lightcone_radius(a))
        counts = _deposit(self.x, self.n, c["ng"], c["box"], c.get("tsc"), self.box is None)
        self.phi = self.solve(self.source(counts, 1.5 * OM / a, 0.0), 0.0)

    def drift(self, coef):
        x = self.x[:, :self.n]
        for d in range(3):
            v = x[d] + self.p[d, :self.n] * coef
            if self.box is None:
                v = torch.where(v < 0.0, v + self.c["box"], v)
                v = torch.where(v >= self.c["box"], v - self.c["box"], v)
            x[d] = v

    def step(self, a, da, resort):
        c, per = self.c, self.box is None
        dtau, am, s, k1, k2 = _scalars(c, a, da)
        if resort:
            self.permute(_sorted_order(self.x, self.n, c), self.n)
        self.drift(0.5 * dtau / a)
        counts = _deposit(self.x, self.n, c["ng"], c["box"], c.get("tsc"), per)
        if c.get("solver") == "ade":
            rhs = self.source(counts, s, 0.0)
            self.phi = _ade(self.phi, rhs, 1.0 / k1, True)
        else:
            self.phi = self.solve(self.source(counts, s, k1), k1)
        g = _force(self.x, self.n, self.phi, c["ng"], c["box"], c.get("tsc"), per)
        self.p[:, :self.n] += (am * dtau) * g
        if not c.get("fp64"):
            self.p = self.p.float().double()      # momenta are stored in 32 bits
        del g
        self.drift(0.5 * dtau / (a + da))
        if c.get("solver") == "ade":
            self.phi = _ade(self.phi, rhs, 1.0 / k2, False)
        elif k2 > 0.0:
            self.phi = self.solve(self.source(counts, s, k2), k2)
        return dtau


def _ade(phi, f, lam, forward):
    """Saul'yev sweep of the periodic mesh, cells of one i + j + k together."""
    n = phi.shape[0]
    i = torch.arange(n, device=DEV)
    t = (i[:, None, None] + i[None, :, None] + i[None, None, :]).reshape(-1)
    order = torch.sort(t, stable=True).indices
    ends = torch.cumsum(torch.bincount(t), 0).tolist()
    u, src = phi.reshape(-1).clone(), f.reshape(-1)
    inv, m, lo = 1.0 / (1.0 + 3.0 * lam), n - 1, 0
    parts = []
    for hi in ends:
        parts.append(order[lo:hi])
        lo = hi
    for q in parts if forward else reversed(parts):
        x, y, z = q & m, (q // n) & m, q // (n * n)
        s = torch.zeros(q.shape, dtype=F64, device=DEV)
        for e in (-1, 1):
            s += u[(z * n + y) * n + ((x + e) & m)]
            s += u[(z * n + ((y + e) & m)) * n + x]
            s += u[((((z + e) & m)) * n + y) * n + x]
        u[q] = ((1.0 - 3.0 * lam) * u[q] + lam * (s - src[q])) * inv
    return u.view(phi.shape)


def _spectrum(x, c):
    ng, npart, box = c["ng"], c["n"], 100.0
    counts = _deposit(x, npart, ng, box, False)
    delta = counts.double() / (npart / ng ** 3 * 2.0 ** (3 * FRAC_BITS)) - 1.0
    dk = torch.fft.fftn(delta) / ng ** 3
    raw = box ** 3 * (dk.real ** 2 + dk.imag ** 2)
    f = torch.fft.fftfreq(ng, 1.0 / ng, device=DEV, dtype=F64).round()
    fx, fy, fz = f[None, None, :], f[None, :, None], f[:, None, None]
    f2 = fx * fx + fy * fy + fz * fz
    shell = torch.round(torch.sqrt(f2)).long()
    nb = ng // 2
    shell[shell > nb] = 0
    shell = shell.reshape(-1)

    def mean(v):
        return torch.bincount(shell, weights=v.expand(ng, ng, ng).reshape(-1),
                              minlength=nb + 1)[1:] / modes

    modes = torch.bincount(shell, minlength=nb + 1)[1:]
    s1 = 1.0 - 2.0 / 3.0 * torch.sin(math.pi * f / ng) ** 2
    c1 = mean(s1[None, None, :] * s1[None, :, None] * s1[:, None, None])
    k = mean(torch.sqrt(f2)) * (2.0 * math.pi / box)
    praw = mean(raw)
    sig = praw - (box ** 3 / npart * c1 if c["shot"] else 0.0)
    p = sig
    if c["jing"]:
        kn, neff = k.cpu().numpy(), np.zeros(nb)
        f2s = f2.clone()
        f2s[0, 0, 0] = 1.0
        m = torch.arange(-2, 3, device=DEV, dtype=F64)
        g = f[:, None] + ng * m[None, :]
        w = torch.sinc(g / ng) ** 4
        for it in range(4):
            ne = torch.cat([torch.zeros(1, dtype=F64), torch.as_tensor(neff)]).to(DEV)
            half = 0.5 * ne[shell].view(ng, ng, ng)
            tot = torch.zeros((ng,) * 3, dtype=F64, device=DEV)
            for a in range(5):
                for b in range(5):
                    for d in range(5):
                        r = (g[None, None, :, a] ** 2 + g[None, :, None, b] ** 2
                             + g[:, None, None, d] ** 2) / f2s
                        r[0, 0, 0] = 1.0
                        tot += (w[None, None, :, a] * w[None, :, None, b] * w[:, None, None, d]
                                * torch.exp(half * torch.log(r)))
            p = sig / mean(tot)
            pn = p.cpu().numpy()
            for b in range(nb):
                lo, hi = max(b - 1, 0), min(b + 1, nb - 1)
                neff[b] = 0.0
                if hi != lo and pn[lo] > 0.0 and pn[hi] > 0.0 and kn[lo] > 0.0:
                    neff[b] = min(max(math.log(pn[hi] / pn[lo]) / math.log(kn[hi] / kn[lo]), -4.0), 4.0)
    return [k, p, praw, None]


_TAPS = [(dx, dy, dz) for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]


def _bf(t):
    return t.to(torch.bfloat16).double()


def _conv(x, w, b=None):
    """x (n, n, n, 16), w (27, 16, 16): sum over taps of x[v + off] w."""
    y = torch.zeros(x.shape[:3] + (w.shape[2],), dtype=F64, device=DEV)
    for t, (dx, dy, dz) in enumerate(_TAPS):
        y += torch.roll(x, (-dz, -dy, -dx), (0, 1, 2)) @ w[t]
    return y if b is None else y + b


def _conv_back(g, w):
    y = torch.zeros(g.shape[:3] + (w.shape[1],), dtype=F64, device=DEV)
    for t, (dx, dy, dz) in enumerate(_TAPS):
        y += torch.roll(g, (dz, dy, dx), (0, 1, 2)) @ w[t].T.contiguous()
    return y


def _train(s):
    n = s.case["ng"]
    v = n ** 3
    w = [q[:27 * 256].view(27, 16, 16).double() for q in s.params.view(5, -1)]
    b = [q[27 * 256:].double() for q in s.params.view(5, -1)]
    x = torch.zeros((n, n, n, 16), dtype=F64, device=DEV)
    x[..., 0] = _bf(s.r * torch.tensor(0.9, dtype=torch.float32))
    x[..., 1] = _bf(s.phi * torch.tensor(1.1, dtype=torch.float32))
    x[..., 2] = float(torch.tensor(0.113).bfloat16())
    acts = [x]
    for l in range(4):
        acts.append(_bf(torch.relu(_conv(acts[-1], _bf(w[l]), b[l])).float()))
    d = _conv(acts[4], _bf(w[4]), b[4])[..., 0] - s.target.double() * float(np.float32(0.8))
    loss = (d * d).mean()
    g = torch.zeros((n, n, n, 16), dtype=F64, device=DEV)
    g[..., 0] = _bf((2.0 * d / v).float())
    grad = [None] * 5
    for l in range(4, -1, -1):
        dw = torch.stack([torch.roll(acts[l], (-dz, -dy, -dx), (0, 1, 2)).reshape(v, 16).T.contiguous()
                          @ g.reshape(v, 16) for dx, dy, dz in _TAPS])
        grad[l] = torch.cat([dw.reshape(-1), g.reshape(v, 16).sum(0)])
        if l:
            g = _bf((_conv_back(g, _bf(w[l])) * (acts[l] > 0)).float())
    frozen = torch.zeros((5, 27 * 256 + 16), dtype=torch.bool, device=DEV)
    frozen[0, :27 * 256].view(27, 16, 16)[:, 3:, :] = True
    frozen[4, :27 * 256].view(27, 16, 16)[:, :, 1:] = True
    frozen[4, 27 * 256 + 1:] = True
    frozen, grad = frozen.reshape(-1), torch.cat(grad)
    m1 = 0.9 * s.m1.double() + 0.1 * grad
    m2 = 0.999 * s.m2.double() + 0.001 * grad * grad
    p = s.params.double() - s.lr * (m1 / (1 - 0.9 ** s.step)) / (torch.sqrt(m2 / (1 - 0.999 ** s.step)) + 1e-8)
    return [torch.where(frozen, torch.zeros_like(p), p), torch.where(frozen, s.m1.double(), m1),
            torch.where(frozen, s.m2.double(), m2), loss.reshape(1)]


def exact(case, seed):
    k, ng = case["kind"], case["ng"]
    if k in ("run", "step", "shrink"):
        x, p = _particles(case["n1d"], case["box"], case["a0"], seed, case.get("fp64", False))
        e = _Exact(case, x, p)
        del x, p
        e.start(case["a0"])
        if k == "run":
            edges = np.linspace(case["a0"], 1.0, case["steps"] + 1)
            for a, b in zip(edges[:-1], edges[1:]):
                e.step(a, b - a, False)
            return [e.x, e.p, e.phi]
        a, da = case["a0"], (1.0 - (0.02 if k == "shrink" else case["a0"])) / case["steps"]
        dtau = e.step(a, da, case["sort_every"] > 0)
        if k == "step":
            return [e.x, e.p, e.phi, None]
        r = _lightcone_radius(a + da)
        m, n0 = e.shrink(r), case["n1d"] ** 3
        x1, p1 = e.x[:, e.n:e.n + m], e.p[:, e.n:e.n + m]
        # |x1 - u v - o| = r + u c dtau at the particle's crossing
        v, o, light = p1 * (dtau / (a + da)), x1 - 0.5 * case["box"], C_LIGHT * dtau
        qa = (v * v).sum(0) - light * light
        qb = -2.0 * (o * v).sum(0) - 2.0 * r * light
        qc = (o * o).sum(0) - r * r
        u = (2.0 * qc / (-qb + torch.sqrt((qb * qb - 4.0 * qa * qc).clamp_min(0.0)))).clamp(0.0, 1.0)
        la = torch.zeros(n0, dtype=F64, device=DEV)
        lx, lp = (torch.zeros((3, n0), dtype=F64, device=DEV) for _ in range(2))
        la[:m], lx[:, :m], lp[:, :m] = a + da - u * da, x1 - u * v, p1
        return [e.x, e.p, e.phi, None, la, lx, lp, None]
    if k == "solve":
        n = case["n"]
        h2 = (100.0 / ng) ** 2
        counts = _deposit(_blobs(n, 100.0, seed), n, ng, 100.0, False)
        rhs = counts.double() * (h2 / (n / ng ** 3 * 2.0 ** (3 * FRAC_BITS))) - h2
        return [_solve(rhs, case["kappa_h2"]), rhs]
    if k == "ade":
        f = _smooth(ng, seed + 7777, 0.01)
        return _ade(_ade(_smooth(ng, seed, 1.0), f, case["lam"], True), f, case["lam"], False)
    if k == "particles":
        x = _blobs(case["n"], 100.0, seed)
        x = x[:, _sorted_order(x, case["n"], dict(case, box=100.0))]
        g = _force(x, case["n"], _smooth(ng, seed, 1.0), ng, 100.0, case["tsc"])
        return [x, torch.ones(x.shape, dtype=F64, device=DEV), None, None, g]
    if k == "pk":
        return _spectrum(_blobs(case["n"], 100.0, seed), case)
    s = prepare(case, seed)
    if k == "train":
        return _train(s)
    shape = (ng, ng, ng, 16)
    w = _bf(s.weight.view(27, 16, 16))
    x, g = (t.view(torch.bfloat16).double().view(shape) for t in (s.inp, s.grad))
    y = torch.relu(_conv(x, w, s.bias.double()))
    return [y.view(-1, 16), (_conv_back(g, w) * (x > 0)).view(-1, 16)]
