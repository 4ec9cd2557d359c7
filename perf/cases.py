"""The work that programs have the phase-space lattice do, as timed cases.

Every case is one call, or one short sequence of calls, of the public
interface on inputs already on the GPU:

  run1d, run2d  a lattice handle advances a state by some steps under
                prestaged flow slices (or, flow "modes", under slices it
                first synthesises from a mode table);
  batch         many independent 1D lattices advanced together;
  coarse        the stride-4 coarse velocity lattice with its learned
                face-flux correction;
  train         Adam steps of the correction network from given weights;
  observe       restriction, moments, density and box statistics of a state;
  s1            the velocity structure function of a state.

Flows are sums of Fourier modes scaled to max |u| = 3 with the velocity
lattice reaching Vmax = 3, and tau_p is set so that the drift CFL of a
collision sub-step is 0.4 whatever the sizes are.  States are local
Maxwellians around 0.6 u with noise in space and in every cell.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_1508_02899_amd import Batch, Lattice, LatticeSpec, Member, Mlp
from paper_1508_02899_amd.coarse import initial_params
from paper_1508_02899_amd.lattice import recommended_pitch, restrict

UMAX = VMAX = 3.0
CFL = 0.4
SPLIT_NV = (17, 33, 65, 129)
RESIDENT, CHUNK = 1, 32  # the batch schedule its own tuner picks
NH = 64  # hidden units of a layer of the network


def listed():
    return [
        # one step of the smallest lattice in use (256 x 33, double): launches
        # and host work are all there is
        dict(name="step-1d-256-v33-f64", kind="run1d", nx=256, nv=33,
             dtype="f64", scheme="koren", nsub=1, steps=1),
        # the same lattice run for 200 steps in a call, a flow slice per step
        dict(name="run-1d-256-v33-f64", kind="run1d", nx=256, nv=33,
             dtype="f64", scheme="koren", nsub=1, steps=200),
        # the paper's finest 1D velocity lattice, long run
        dict(name="run-1d-16384-v129", kind="run1d", nx=16384, nv=129,
             dtype="f32", scheme="koren", nsub=1, steps=100),
        # the flagship 2D run, its flow synthesised on the device
        dict(name="run-2d-512-v33", kind="run2d", nx=512, ny=512, nv=33,
             dtype="f32", scheme="koren", nsub=1, steps=8, flow="modes",
             kmax=32),
        # the fine lattice of the coarse-model workflow: short Stokes times
        # need several collision sub-steps per streaming step
        dict(name="fine-2d-256-v65-nsub4", kind="run2d", nx=256, ny=256,
             nv=65, dtype="f32", scheme="koren", nsub=4, steps=2,
             flow="given", kmax=32),
        # a ragged medium lattice with the first-order scheme
        dict(name="ragged-2d-210x150-v13-upwind", kind="run2d", nx=210,
             ny=150, nv=13, dtype="f32", scheme="upwind", nsub=1, steps=16,
             flow="given", kmax=12),
        # double precision in 2D (accuracy references)
        dict(name="run-2d-192-v17-f64", kind="run2d", nx=192, ny=192, nv=17,
             dtype="f64", scheme="koren", nsub=1, steps=8, flow="given",
             kmax=16),
        # 256 independent 1D realizations advanced together
        dict(name="batch-256x1d", kind="batch", count=256, nx_lo=512,
             nx_hi=8192, nvs="33,65,129", steps=10, hold=5),
        # the coarse lattice with the learned correction
        dict(name="coarse-mlp-256", kind="coarse", nx=256, ny=256, steps=4,
             nsub=1, eps=8e-3),
        # one epoch of the network's a-priori training
        dict(name="train-8192x24", kind="train", batch=8192, steps=24),
        # observables of a fine state and its restriction
        dict(name="observe-2d-128-v65", kind="observe", nx=128, ny=128,
             nv=65, levels=8),
        # structure function of a 2D state at six separations
        dict(name="s1-2d-256-v17", kind="s1", nx=256, ny=256, nv=17, nr=6),
    ]


def _spread(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["run1d", "run1d", "run2d", "run2d", "run2d", "batch",
                       "coarse", "train", "observe", "s1"])
    scheme = rng.choice(["koren", "koren", "koren", "upwind"])
    if kind == "run1d":
        dtype = rng.choice(["f32", "f32", "f64"])
        nv = rng.choice([5, 9, 17, 21, 33, 45, 65] +
                        ([129] if dtype == "f32" else []))
        return dict(kind=kind, nx=_spread(rng, 64, 40000), nv=nv, dtype=dtype,
                    scheme=scheme, nsub=rng.choice([1, 1, 2, 3]),
                    steps=_spread(rng, 1, 100))
    if kind == "run2d":
        dtype = rng.choice(["f32", "f32", "f32", "f64"])
        nv = rng.choice([5, 9, 17, 33] if dtype == "f64" else
                        [5, 9, 13, 17, 21, 33, 65])
        nsub = rng.choice([1, 1, 2, 3, 5])
        cap = 4e8 if dtype == "f32" else 1.2e8  # cell updates of a pass
        most = math.sqrt(cap / (nv * nv * nsub))
        nx = _spread(rng, 40, min(512, 1.5 * most))
        ny = _spread(rng, 40, min(512, max(41, cap / (nv * nv * nsub * nx))))
        room = cap / (nv * nv * nsub * nx * ny)
        return dict(kind=kind, nx=nx, ny=ny, nv=nv, dtype=dtype,
                    scheme=scheme, nsub=nsub,
                    steps=max(1, _spread(rng, 1, max(1.0, min(16.0, room)))),
                    flow=rng.choice(["given", "modes"]),
                    kmax=rng.randint(4, 18))
    if kind == "batch":
        hi = rng.choice([700, 3000, 8192])
        return dict(kind=kind, count=_spread(rng, 4, 200), nx_lo=64,
                    nx_hi=hi, steps=rng.randint(2, 8), hold=rng.randint(1, 8),
                    nvs=rng.choice(["33,65,129", "17,33", "9,21,45",
                                    "33,65,129"]))
    if kind == "coarse":
        return dict(kind=kind, nx=_spread(rng, 40, 256),
                    ny=_spread(rng, 40, 256), steps=rng.randint(1, 4),
                    nsub=rng.choice([1, 2, 4]),
                    eps=rng.choice([0.0, 8e-3, 2.4e-2]))
    if kind == "train":
        return dict(kind=kind, batch=_spread(rng, 500, 16384),
                    steps=rng.randint(4, 24))
    if kind == "observe":
        levels = rng.randint(3, 6)
        tile = 2 ** (levels - 1)
        return dict(kind=kind, nx=tile * rng.randint(64 // tile, 160 // tile),
                    ny=tile * rng.randint(64 // tile, 160 // tile),
                    nv=rng.choice([9, 17, 33, 65]), levels=levels)
    return dict(kind="s1", nx=_spread(rng, 40, 256), ny=_spread(rng, 40, 256),
                nv=rng.choice([9, 13, 17]), nr=rng.randint(2, 8))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _rand(shape, g, dtype=torch.float32):
    return torch.rand(shape, generator=g, device="cuda", dtype=dtype)


def _geometry(case):
    """dx, dt, tau_p, kappa of a lattice case (vstride 4 for the coarse
    lattice, whose time step is that of the 65-velocity fine one)."""
    stride = 4 if case["kind"] == "coarse" else 1
    nv = case.get("nv", 17)
    dx = 2 * math.pi / case["nx"]
    dv = VMAX / ((nv - 1) // 2)
    dt = stride * dx / dv
    dts = dt / case.get("nsub", 1)
    tau = (dts / dv) * (UMAX + VMAX) / CFL
    return dx, dv, dt, tau, min(1e-4, 0.2 * dv * dv / dts)


def _modes2d(g, slices, kmax):
    """Streamfunction mode table [slices, 2K+1, K+1, 2] (float64), shell
    spectrum k^-3, the phases turning from slice to slice."""
    ky = torch.arange(-kmax, kmax + 1, device="cuda", dtype=torch.float64)
    kx = torch.arange(0, kmax + 1, device="cuda", dtype=torch.float64)
    k = torch.sqrt(ky[:, None] ** 2 + kx[None, :] ** 2)
    amp = torch.where((k >= 1) & (k <= kmax), k.clamp(min=1.0) ** -3.0,
                      torch.zeros_like(k))
    a = torch.randn(k.shape, generator=g, device="cuda", dtype=torch.float64)
    ph = 2 * math.pi * _rand(k.shape, g, torch.float64)
    w = torch.randn(k.shape, generator=g, device="cuda", dtype=torch.float64)
    s = torch.arange(slices, device="cuda", dtype=torch.float64)[:, None, None]
    th = ph + 0.05 * s * w
    return torch.stack([amp * a * torch.cos(th), amp * a * torch.sin(th)], -1)


def _flow2d(coef, nx, ny, dx):
    """u [slices, 2, ny, nx] in float64 of a 2D mode table."""
    c = torch.view_as_complex(coef.double().contiguous())
    K = c.shape[2] - 1
    kx = torch.arange(K + 1, device="cuda", dtype=torch.float64)
    ky = torch.arange(-K, K + 1, device="cuda", dtype=torch.float64)

    def turns(k, n):
        p = torch.remainder(k[:, None] * torch.arange(
            n, device="cuda", dtype=torch.float64)[None, :], n)
        return torch.polar(torch.ones_like(p), 2 * math.pi * p / n)

    ex, ey = turns(kx, nx), turns(ky, ny)
    gx, gy = 2 * math.pi / (nx * dx), 2 * math.pi / (ny * dx)
    out = torch.empty((c.shape[0], 2, ny, nx), device="cuda",
                      dtype=torch.float64)
    for s in range(c.shape[0]):
        a = c[s] @ ex
        b = (c[s] * (-1j * gx * kx)[None, :]) @ ex
        out[s, 0] = ((ey * (1j * gy * ky)[:, None]).T @ a).real
        out[s, 1] = (ey.T @ b).real
    return out


def _flow1d(g, slices, nx, modes=16):
    """u [slices, 1, nx] in float64, amplitudes 1/k."""
    k = torch.arange(1, modes + 1, device="cuda", dtype=torch.float64)
    x = torch.arange(nx, device="cuda", dtype=torch.float64)
    p = 2 * math.pi * torch.remainder(k[:, None] * x[None, :], nx) / nx
    amp = torch.randn(modes, generator=g, device="cuda",
                      dtype=torch.float64) / k
    ph = 2 * math.pi * _rand((modes,), g, torch.float64)
    w = torch.randn(modes, generator=g, device="cuda", dtype=torch.float64)
    s = torch.arange(slices, device="cuda", dtype=torch.float64)
    th = ph[None, :] + 0.05 * s[:, None] * w[None, :]
    u = (amp * torch.cos(th)) @ torch.cos(p) - (amp * torch.sin(th)) @ \
        torch.sin(p)
    return (u * (UMAX / u.abs().max()))[:, None, :]


def _state(g, case, u0, dv, out=None):
    """A state [nv^dim, ny, nx] ([nv, nx] in 1D) around 0.6 u0, unit mass
    density on average; u0 [dim, ...sites]."""
    dim, nv = u0.shape[0], case.get("nv", 17)
    dtype = torch.float64 if case.get("dtype") == "f64" else torch.float32
    h = (nv - 1) // 2
    v = (torch.arange(nv, device="cuda", dtype=dtype) - h) * dv
    sites = u0.shape[1:]
    rho = 0.5 + _rand(sites, g, dtype)
    lines = [torch.exp(-(v.view(-1, *([1] * len(sites))) -
                         0.6 * u0[k].to(dtype)) ** 2 / (2 * 0.7 ** 2))
             for k in range(dim)]
    lines = [a / (a.sum(0) * dv) for a in lines]
    if out is None:
        out = torch.empty((nv ** dim, *sites), device="cuda", dtype=dtype)
    for j in range(nv if dim == 2 else 1):
        row = lines[0] * rho if dim == 1 else lines[0] * (lines[1][j] * rho)
        out[j * nv:(j + 1) * nv] = row * (0.8 + 0.4 * _rand(row.shape, g,
                                                            dtype))
    return out


def _lattice_inputs(case, seed):
    """(flow table or None, u float64 or None when the table is scaled, g)."""
    g = _gen(seed)
    dx = 2 * math.pi / case["nx"]
    if case["kind"] == "run1d":
        return None, _flow1d(g, case["steps"], case["nx"]), g
    K = min(case.get("kmax", 16), (min(case["nx"], case["ny"]) - 1) // 2)
    slices = case.get("steps", 1)
    coef = _modes2d(g, slices, K)
    u = _flow2d(coef, case["nx"], case["ny"], dx)
    scale = UMAX / u.abs().max()
    if case.get("flow") == "modes":
        coef = (coef * scale * 0.999).float()
        return coef, _flow2d(coef, case["nx"], case["ny"], dx), g
    return None, u * scale, g


def _spec(case):
    dx = _geometry(case)[0]
    two = case["kind"] != "run1d"
    spec = LatticeSpec(dim=2 if two else 1, nx=case["nx"],
                       ny=case["ny"] if two else 1, nv=case.get("nv", 17),
                       dx=dx, vstride=4 if case["kind"] == "coarse" else 1,
                       scheme=case.get("scheme", "koren"),
                       dtype=case.get("dtype", "f32"),
                       nsub=case.get("nsub", 1), u_hold=1)
    if case["kind"] == "run2d":
        spec.plane_pitch = recommended_pitch(spec)
    return spec


def _net(seed):
    """Weights of a trained network's size (the initial weights with a
    larger output layer and biases)."""
    rng = np.random.default_rng(int(seed))
    p = initial_params(int(seed), out_scale=0.05)
    p += (0.05 * rng.standard_normal(p.size)).astype(np.float32)
    p[4736:] *= 0.2
    return p


def _shapes(case):
    r = random.Random(f"{case['count']}|{case['nx_lo']}|{case['nx_hi']}|"
                      f"{case['nvs']}")
    nvs = [int(x) for x in case["nvs"].split(",")]
    return [(r.randint(case["nx_lo"], case["nx_hi"]), r.choice(nvs))
            for _ in range(case["count"])]


def _members(case):
    out = []
    for nx, nv in _shapes(case):
        dx, _, dt, tau, kappa = _geometry(dict(kind="run1d", nx=nx, nv=nv))
        out.append(Member(nx=nx, nv=nv, dx=dx, dt=dt, tau_p=tau, kappa=kappa,
                          u_hold=case["hold"],
                          n_u_slices=-(-case["steps"] // case["hold"])))
    return out


def _member_inputs(case, seed):
    """Per member (state [nv, nx], u [slices, 1, nx]) in float32."""
    g = _gen(seed)
    out = []
    for m in _members(case):
        u = _flow1d(g, m.n_u_slices, m.nx, 8).float()
        dv = VMAX / ((m.nv - 1) // 2)
        out.append((_state(g, dict(nv=m.nv), u[0], dv), u))
    return out


def _samples(case, seed):
    """Training samples: stencils of smooth positive profiles, drift, ln St,
    targets a smooth function of them with noise."""
    g = _gen(seed)
    n = case["batch"] * case["steps"]
    X = torch.zeros((n, 8), device="cuda")
    s = torch.exp(-0.5 * ((torch.arange(5, device="cuda") - 2 +
                           1.5 * torch.randn((n, 1), generator=g,
                                             device="cuda")) /
                          (0.5 + 1.5 * _rand((n, 1), g))) ** 2) + 1e-3
    X[:, :5] = s / s.sum(1, keepdim=True)
    X[:, 5] = 0.4 * _rand((n,), g)
    X[:, 6] = math.log(2.0)
    t = 0.05 * X[:, 5] * (X[:, 0] - X[:, 3]) + 0.01 * torch.randn(
        n, generator=g, device="cuda")
    return X, t, 0.01 + _rand((n,), g)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        return dict(case=case, mlp=Mlp(), p0=_net(seed),
                    data=_samples(case, seed))
    if kind == "batch":
        b = Batch(_members(case))
        if all(nv in SPLIT_NV for _, nv in _shapes(case)):
            b.schedule(RESIDENT, 0, CHUNK)
        f = torch.zeros(b.total_elems, device="cuda")
        u = torch.empty(b.total_u, device="cuda")
        for m, fo, uo, p, (s, w) in zip(b.members, b.f_off, b.u_off, b.pitch,
                                        _member_inputs(case, seed)):
            f[fo:fo + m.nv * p].view(m.nv, p)[:, :m.nx] = s
            u[uo:uo + w.numel()] = w.flatten()
        return dict(case=case, batch=b, f=f, u=u)
    spec = _spec(case)
    coef, u, g = _lattice_inputs(case, seed)
    dx, dv, dt, tau, kappa = _geometry(case)
    lat = Lattice(spec)
    f = _state(g, case, u[0], dv, spec.empty_state())
    st = dict(case=case, lat=lat, f=f, dt=dt, tau=tau, kappa=kappa, coef=coef,
              u=u.to(f.dtype).contiguous())
    if kind == "coarse":
        st["mlp"] = Mlp()
        st["mlp"].set_params(_net(seed))
        st["mlp"].attach(lat, 2.0, case["eps"])
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "train":
        mlp = state["mlp"]
        mlp.set_params(state["p0"])
        loss = mlp.train(*state["data"], batch=case["batch"],
                         steps=case["steps"], lr=1e-3)
        return dict(params=mlp.get_params(), loss=np.float32(loss))
    if kind == "batch":
        state["batch"].step(state["f"], state["u"], case["steps"])
        return state["f"]
    lat, f = state["lat"], state["f"]
    if kind == "observe":
        m = lat.moments(f, state["dt"])
        rho = lat.density(f, state["dt"])
        return dict(restricted=restrict(f, 2), rho=rho,
                    moments=np.array([m["mass"], *m["second_moment"],
                                      m["variance"]]),
                    rho_r2=lat.rho_r2(rho, case["levels"]))
    if kind == "s1":
        return lat.s1(f, state["dt"], _separations(case))
    u = state["u"]
    if state["coef"] is not None:
        u = lat.flow_from_modes(state["coef"])
    lat.step(f, u, state["tau"], state["kappa"], state["dt"], case["steps"])
    return f if state["coef"] is None else (f, u)


def _separations(case):
    top = min(case["nx"], case["ny"]) // 4
    return sorted({min(top, 2 ** k) if k else 0 for k in
                   range(1, case["nr"] + 1)})


def work(case):
    kind = case["kind"]
    if kind == "train":  # forward and twice as much backward, every sample
        n = case["batch"] * case["steps"]
        return dict(bytes=40.0 * n + 2 * 4 * 4801,
                    flops=3.0 * 2 * n * (8 * NH + NH * NH + NH))
    if kind == "batch":
        cells = sum(nx * nv for nx, nv in _shapes(case))
        sites = sum(nx for nx, _ in _shapes(case))
        sl = -(-case["steps"] // case["hold"])
        return dict(bytes=8.0 * cells * case["steps"] + 4.0 * sites * sl,
                    flops=25.0 * cells * case["steps"])
    el = 8 if case.get("dtype") == "f64" else 4
    dim = 1 if kind == "run1d" else 2
    sites = case["nx"] * case.get("ny", 1)
    nv = case.get("nv", 17)
    cells = sites * nv ** dim
    if kind == "observe":
        nvc = (nv - 1) // 4 + 1
        return dict(bytes=4.0 * cells + 4.0 * sites * nvc ** 2 + 8.0 * sites,
                    flops=12.0 * cells)
    if kind == "s1":
        return dict(bytes=4.0 * cells,
                    flops=2.0 * cells * nv * nv +
                    4.0 * cells * len(_separations(case)))
    steps, nsub = case["steps"], case["nsub"]
    flops = (25.0 if dim == 1 else 50.0) * cells * steps * nsub
    if kind == "coarse":  # the faces of every site through the network
        flops += 2.0 * steps * sites * 544 * (8 * NH + NH * NH + NH)
    return dict(bytes=steps * (2.0 * cells + dim * sites) * el, flops=flops)


# ------------------------------------------------------------ in 64 bits
def _median0(a, b):
    """The median of a, b and 0."""
    return torch.maximum(torch.minimum(a, b), torch.minimum(
        torch.maximum(a, b), torch.zeros_like(a)))


def _limited(dp, dm):
    return _median0(dp, _median0(dm / 6 + dp / 3, dm))


def _face_flux(c, nu, koren):
    """Drift fluxes through the inner faces of axis 0 (cells k-1 | k)."""
    z = torch.zeros_like(c[:1])
    gp, gm = nu.clamp(min=0) * c, nu.clamp(max=0) * c
    fl = gp[:-1] + gm[1:]
    if koren:
        dp = torch.cat([z, gp])
        dp = dp[1:] - dp[:-1]          # gp[k] - gp[k-1], gp[-1] = 0
        dm = torch.cat([gm, z])
        dm = dm[:-1] - dm[1:]          # gm[k] - gm[k+1], gm[nv] = 0
        fl = fl + _limited(dp[1:], dp[:-1]) + _limited(dm[:-1], dm[1:])
    return fl


def _apply(c, fl):
    c = c.clone()
    c[:-1] -= fl
    c[1:] += fl
    return c


def _exact_collide(c, u, h, alpha, beta, D, koren):
    """One collision sub-step of c [nvy, nvx, ny, nx] (1D: [1, nv, 1, nx]);
    u [dim, ny, nx]."""
    nvx = c.shape[1]
    v = torch.arange(nvx, device=c.device, dtype=c.dtype) - h
    v = v.view(-1, 1, 1)
    two = u.shape[0] == 2
    for k in range(2 if two else 1):
        nu = (alpha * u[k][None] - beta * v)[:, None]
        a = c if k else c.transpose(0, 1)
        a = _apply(a, _face_flux(a, nu, koren))
        c = a if k else a.transpose(0, 1)
    for k in range(2 if two else 1):
        a = c if k else c.transpose(0, 1)
        a = _apply(a, D * (a[:-1] - a[1:]))
        c = a if k else a.transpose(0, 1)
    return c


def _exact_run(f, us, case, geo, stride=1, after=None):
    """f [nv^dim, ...] advanced under us [steps, dim, ny, nx], in float64;
    after(c, u): what follows each step."""
    dx, dv, dt, tau, kappa = geo
    nv = case.get("nv", 17)
    h, nsub = (nv - 1) // 2, case.get("nsub", 1)
    two = f.dim() == 3
    ny, nx = (f.shape[1], f.shape[2]) if two else (1, f.shape[1])
    c = f.double().reshape(nv if two else 1, nv, ny, nx)
    dts = dt / nsub
    j = torch.arange(nv, device="cuda")[:, None] - h
    ix = (torch.arange(nx, device="cuda")[None, :] - stride * j) % nx
    iy = (torch.arange(ny, device="cuda")[None, :] - stride * j) % ny
    for s in range(us.shape[0]):
        u = us[s].double().reshape(-1, ny, nx)
        c = c.gather(3, ix[None, :, None, :].expand(c.shape[0], nv, ny, nx))
        if two:
            c = c.gather(2, iy[:, None, :, None].expand(nv, nv, ny, nx))
        for _ in range(nsub):
            c = _exact_collide(c, u, h, dts / (dv * tau), dts / tau,
                               kappa * dts / (dv * dv),
                               case.get("scheme", "koren") == "koren")
        if after is not None:
            c = after(c, u)
    return c.reshape(f.shape)


def _gelu(z):
    s = torch.sigmoid(2 * math.sqrt(2 / math.pi) * (z + 0.044715 * z ** 3))
    return z * s, s


def _layers(p):
    p = torch.as_tensor(p, device="cuda").double()
    o = [512, 64, 4096, 64, 64, 1]
    w1, b1, w2, b2, w3, b3 = torch.split(p, o)
    return w1.view(8, 64), b1, w2.view(64, 64), b2, w3, b3


def _exact_correction(c, u, p, geo, eps):
    """The learned face fluxes applied to c [17, 17, ny, nx] (weights as
    rounded to bfloat16, everything else in float64)."""
    dx, dv, dt, tau, _ = geo
    q = torch.as_tensor(p, device="cuda")
    w1, b1, w2, b2, w3, b3 = _layers(q)
    w1, w2, w3 = (w.bfloat16().double() for w in (w1, w2, w3))
    M = c.sum((0, 1))
    new = c.clone()
    for ax in range(2):
        a = c.transpose(0, 1) if ax == 0 else c   # faces along axis 0
        z = torch.zeros((3, *a.shape[1:]), device="cuda", dtype=c.dtype)
        pad = torch.cat([z, a, z])
        G = torch.empty((16, *a.shape[1:]), device="cuda", dtype=c.dtype)
        for k in range(1, 17):
            nu = dt / (tau * dv) * (u[ax] - (k - 0.5 - 8) * dv)
            up = (nu >= 0)[None]
            st = [torch.where(up, pad[k + i], pad[k + 5 - i])
                  for i in range(5)]
            ms = sum(st)
            use = (ms > 1e-30) & (ms >= eps * M[None])
            x = torch.stack([s / torch.where(use, ms, torch.ones_like(ms))
                             for s in st], -1)
            more = torch.stack([nu.abs().expand(ms.shape),
                                torch.full_like(ms, math.log(2.0))], -1)
            x = torch.cat([x, more], -1)
            y = _gelu(_gelu(x @ w1[:7] + b1)[0] @ w2 + b2)[0] @ w3 + b3
            g = torch.where(up, ms * y, -ms * y)
            cap = 0.25 * torch.where(g > 0, a[k - 1], a[k])
            g = torch.maximum(torch.minimum(g, cap), -cap)
            G[k - 1] = torch.where(use, g, torch.zeros_like(g))
        d = torch.zeros_like(a)
        d[:-1] -= G
        d[1:] += G
        new += d.transpose(0, 1) if ax == 0 else d
    return new


def _exact_train(p, data, batch, steps, lr):
    """Adam on the weighted square error, weights and layer inputs rounded
    to bfloat16 (straight through), everything else in float64."""
    X, t, w = (a.double() for a in data)

    def qb(a):
        return a.float().bfloat16().double()

    p = torch.as_tensor(p, device="cuda").double()
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    mean = w.mean()
    loss = None
    for k in range(steps):
        x, tt, ww = (a[k * batch:(k + 1) * batch] for a in (X, t, w))
        w1, b1, w2, b2, w3, b3 = _layers(p)
        x = qb(x)
        z1 = x @ qb(w1) + b1
        h1, s1 = _gelu(z1)
        h1 = qb(h1)
        z2 = h1 @ qb(w2) + b2
        h2, s2 = _gelu(z2)
        h2 = qb(h2)
        e = h2 @ qb(w3) + b3 - tt
        loss = (ww * e * e).sum() / (batch * mean)
        dy = 2 * ww * e / (batch * mean)

        def slope(z, s):
            return s + 2 * math.sqrt(2 / math.pi) * z * s * (1 - s) * (
                1 + 3 * 0.044715 * z * z)

        d2 = dy[:, None] * qb(w3) * slope(z2, s2)
        d1 = (d2 @ qb(w2).T) * slope(z1, s1)
        g = torch.cat([(x.T @ d1).flatten(), d1.sum(0), (h1.T @ d2).flatten(),
                       d2.sum(0), h2.T @ dy, dy.sum()[None]])
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - lr * (m / (1 - 0.9 ** (k + 1))) / (
            torch.sqrt(v / (1 - 0.999 ** (k + 1))) + 1e-8)
    return dict(params=p, loss=loss)


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(_net(seed), _samples(case, seed), case["batch"],
                            case["steps"], 1e-3)
    if kind == "batch":
        out = []
        for s, u in _member_inputs(case, seed):
            nv, nx = s.shape
            c = dict(kind="run1d", nx=nx, nv=nv)
            us = u.repeat_interleave(case["hold"], 0)[:case["steps"]]
            # planes lie a multiple of 64 elements apart
            out.append(torch.nn.functional.pad(
                _exact_run(s, us, c, _geometry(c)),
                (0, -nx % 64)).flatten())
        return torch.cat(out)
    coef, u, g = _lattice_inputs(case, seed)
    geo = _geometry(case)
    f = _state(g, case, u[0], geo[1])
    if kind == "observe":
        dv, dx, nv = geo[1], geo[0], case["nv"]
        c = f.double().view(nv, nv, case["ny"], case["nx"])
        nvc = (nv - 1) // 4 + 1
        R = torch.zeros((nvc, nv), device="cuda", dtype=torch.float64)
        for J in range(nvc):
            for o in range(-2, 3):
                if 0 <= 4 * J + o < nv:
                    R[J, 4 * J + o] = 0.125 if abs(o) == 2 else 0.25
        r = torch.tensordot(R, torch.tensordot(R, c, dims=([1], [0])),
                            dims=([1], [1])).transpose(0, 1)
        rho = c.sum((0, 1)) * dv * dv
        ps = c.sum((2, 3))
        v = (torch.arange(nv, device="cuda", dtype=torch.float64) -
             (nv - 1) // 2) * dv
        M, wt = ps.sum(), dx * dx * dv * dv
        qx, qy = (ps.sum(0) * v * v).sum(), (ps.sum(1) * v * v).sum()
        px, py = (ps.sum(0) * v).sum(), (ps.sum(1) * v).sum()
        box, out = rho, []
        for k in range(case["levels"]):
            if k:
                box = box.reshape(box.shape[0] // 2, 2, box.shape[1] // 2,
                                  2).sum((1, 3))
            out.append(box.numel() * (box * box).sum() / box.sum() ** 2)
        return dict(restricted=r.reshape(nvc * nvc, *rho.shape), rho=rho,
                    moments=torch.stack([
                        wt * M, wt * qx, wt * qy,
                        (qx + qy) / M - (px * px + py * py) / (M * M)]),
                    rho_r2=torch.stack(out))
    if kind == "s1":
        nv = case["nv"]
        c = f.double().view(nv * nv, case["ny"], case["nx"])
        j = torch.arange(nv * nv, device="cuda")
        dy, dxv = j // nv, j % nv
        dist = torch.sqrt(((dy[:, None] - dy) ** 2 +
                           (dxv[:, None] - dxv) ** 2).double())
        hh = (dist @ c.reshape(nv * nv, -1)).view_as(c)
        rho = c.sum(0)
        out = []
        for r in _separations(case):
            est = [geo[1] * (c * hh.roll(-r, d)).sum() /
                   (rho * rho.roll(-r, d - 1)).sum() for d in (1, 2)]
            out.append(0.5 * (est[0] + est[1]))
        return torch.stack(out)
    if coef is None:
        us = u.to(f.dtype)
        if kind == "coarse":
            p = _net(seed)
            return _exact_run(
                f, us, case, geo, 4, lambda c, w: _exact_correction(
                    c, w, p, geo, case["eps"]))
        return _exact_run(f, us, case, geo)
    return _exact_run(f, u, case, geo), u
