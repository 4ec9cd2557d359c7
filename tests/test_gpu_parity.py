"""GPU parity: the HIP lattice update against the FP64 oracle.

Same seeded inputs on both sides (the oracle gets the FP32-rounded values
cast to FP64).  Bounds: relative L2 <= 1e-5 for FP32 state, <= 1e-12 for
FP64 state, bit-exact for pure streaming.  Sizes span several tiles and a
ragged tail (nx not a multiple of the 256-lane block or of the 2D
wavefront tile).
"""
import math

import numpy as np
import pytest

from helpers import (FP32_REL_L2, FP64_REL_L2, make_case, rel_l2, run_gpu,
                     run_oracle, say)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv", [3, 5, 9, 17, 33, 65, 129])
@pytest.mark.parametrize("scheme", ["koren", "upwind"])
def test_1d_f32_parity(nv, scheme):
    say(f"1d f32 nv={nv} {scheme}")
    f0, u, p = make_case(1, 300, nv, seed=nv, scheme=scheme)
    got = run_gpu(f0, u, p, 12)
    want = run_oracle(f0, u, p, 12)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2


@pytest.mark.parametrize("nx,nv", [(1, 17), (7, 33), (31, 65), (45, 129),
                                   (64, 33), (65, 17), (1000, 129)])
def test_1d_split_column_short_and_ragged(nx, nv):
    """The split-column 1D pass on lattices shorter than one workgroup's
    sites and with ragged tails; nsub = 3 and stride 4 on the way."""
    say(f"1d split-column nx={nx} nv={nv}")
    f0, u, p = make_case(1, nx, nv, seed=300 + nx + nv, slices=2, s=4,
                         nsub=3)
    got = run_gpu(f0, u, p, 6, u_hold=3)
    want = run_oracle(f0, u, p, 6, u_hold=3)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2


@pytest.mark.parametrize("scheme", ["koren", "upwind"])
def test_1d_long_lattice_one_lane_per_site(scheme):
    """Past 2^19 sites the 1D pass gives each site one lane (the whole
    column in registers); nx = 2^19 + 37 with 33 velocities."""
    nx = (1 << 19) + 37
    say(f"1d one-lane-per-site nx={nx} nv=33 {scheme}")
    f0, u, p = make_case(1, nx, 33, seed=401, scheme=scheme)
    got = run_gpu(f0, u, p, 3)
    want = run_oracle(f0, u, p, 3)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2


@pytest.mark.parametrize("nv", [3, 9, 17, 33, 65])
@pytest.mark.parametrize("scheme", ["koren", "upwind"])
def test_1d_f64_parity(nv, scheme):
    say(f"1d f64 nv={nv} {scheme}")
    f0, u, p = make_case(1, 257, nv, seed=100 + nv, dtype="f64", scheme=scheme)
    got = run_gpu(f0, u, p, 10, dtype="f64")
    want = run_oracle(f0, u, p, 10)
    assert rel_l2(got, want) <= FP64_REL_L2


def test_1d_f64_256x33_1000_steps_renewed_flow():
    """1D periodic 256 x 33 in FP64, random 8-mode flow renewed every 50
    steps (u_hold = 50), St = 1, kappa = 1e-3, 1000 steps, Koren."""
    from paper_1508_02899_amd import inputs
    say("1d f64 256x33, 1000 steps, u_hold 50")
    nx, nv, L = 256, 33, 2 * math.pi
    nsteps, hold = 1000, 50
    u = inputs.flow1d(nx, L, nsteps // hold, modes=8, spectrum="k-1",
                      renew=hold, seed=inputs.seed_for(1), dtype=np.float64)
    tau_p = 1.0 * L  # St = tau_p u_rms / L = 1
    vmax = 5.0
    h = (nv - 1) // 2
    dv = vmax / h
    dx = L / nx
    dt = dx / dv
    f0 = inputs.gaussian_ic(1, nx, nv, dx, dv, dtype=np.float64)
    p = dict(dim=1, dx=dx, dt=dt, tau_p=tau_p, kappa=1e-3, s=1, nsub=1,
             scheme="koren")
    got = run_gpu(f0, u, p, nsteps, dtype="f64", u_hold=hold)
    want = run_oracle(f0, u, p, nsteps, u_hold=hold)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP64_REL_L2


@pytest.mark.parametrize("nv", [3, 5, 7, 9, 11, 13, 15, 17, 19, 21, 25, 33])
def test_2d_f32_parity_koren(nv):
    say(f"2d f32 nv={nv} koren")
    f0, u, p = make_case(2, 70, nv, ny=9, seed=200 + nv)
    got = run_gpu(f0, u, p, 4)
    want = run_oracle(f0, u, p, 4)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2


@pytest.mark.parametrize("nv", [5, 17, 33])
def test_2d_f32_parity_upwind(nv):
    say(f"2d f32 nv={nv} upwind")
    f0, u, p = make_case(2, 45, nv, ny=7, seed=300 + nv, scheme="upwind")
    got = run_gpu(f0, u, p, 4)
    want = run_oracle(f0, u, p, 4)
    assert rel_l2(got, want) <= FP32_REL_L2


def test_2d_f32_parity_nv65():
    say("2d f32 nv=65 koren")
    f0, u, p = make_case(2, 37, 65, ny=5, seed=465)
    got = run_gpu(f0, u, p, 3)
    want = run_oracle(f0, u, p, 3)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2


def _vy_drift_case(nv, flow, nx, ny, seed, dtype):
    """A state with a chosen vertical flow u_y, which sets where the vy drift
    nu(t) = (dt/tau_p)(u_y/dv - (t - h)) changes sign along the rows t: the
    2D pass skips the split half of that drift that is zero on a whole
    wavefront, in loops chosen by that sign change."""
    from paper_1508_02899_amd import inputs
    rng = np.random.default_rng(seed)
    npdt = np.float64 if dtype == "f64" else np.float32
    f0 = inputs.random_state(rng, (nv * nv, ny, nx), npdt)
    L, dt = 2 * math.pi, 0.05
    dx = L / nx
    h = (nv - 1) // 2
    dv = dx / dt
    vmax = h * dv
    ux = 0.5 * np.tanh(rng.standard_normal((ny, nx)))
    uy = {
        # sign change at a row a little past the middle / before it, the
        # same for every site
        "up": np.full((ny, nx), 0.3 * vmax),
        "down": np.full((ny, nx), -0.3 * vmax),
        # a different row for each wavefront of a workgroup
        "wave": 0.5 * vmax * np.sin(2 * math.pi * np.arange(nx) / nx)
        * np.ones((ny, 1)),
        # past either end of the velocity axis: one half is zero throughout
        "beyond": np.full((ny, nx), 1.2 * vmax),
        "below": np.full((ny, nx), -1.2 * vmax),
        # no drag at all (tau_p infinite): both halves are zero
        "nodrag": np.zeros((ny, nx)),
    }[flow]
    u = np.stack([ux, uy])[None].astype(npdt)
    umax = float(np.abs(u).max())
    tau_p = math.inf if flow == "nodrag" else (dt / dv) * (umax + vmax) / 0.4
    kappa = 0.2 * 0.5 * dv * dv / dt
    p = dict(dim=2, dx=dx, dt=dt, tau_p=tau_p, kappa=kappa, s=1, nsub=1,
             scheme="koren")
    return f0, u, p


@pytest.mark.parametrize("flow", ["up", "down", "wave", "beyond", "below",
                                  "nodrag"])
@pytest.mark.parametrize("nv", [17, 33, 65])
def test_2d_vy_drift_half_skipped_where_zero(nv, flow):
    """Each skip mode of the streamed vy drift, and the moves between them
    at the same or at different rows across the wavefronts of a workgroup,
    against the oracle (which always computes both split halves); 300
    sites per row: several workgroups, interior and edge tiles, a ragged
    tail."""
    ny = 3 if nv == 65 else 4
    say(f"2d vy-drift skip nv={nv} flow={flow}")
    f0, u, p = _vy_drift_case(nv, flow, 300, ny, 700 + nv, "f32")
    got = run_gpu(f0, u, p, 3)
    want = run_oracle(f0, u, p, 3)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2
    assert np.isfinite(got).all()


@pytest.mark.parametrize("flow", ["up", "wave", "below"])
def test_2d_vy_drift_half_skipped_f64(flow):
    say(f"2d f64 vy-drift skip nv=33 flow={flow}")
    f0, u, p = _vy_drift_case(33, flow, 200, 3, 800, "f64")
    got = run_gpu(f0, u, p, 3, dtype="f64")
    want = run_oracle(f0, u, p, 3)
    assert rel_l2(got, want) <= FP64_REL_L2


@pytest.mark.parametrize("nx,ny,nv", [(1, 1, 9), (1, 5, 33), (7, 1, 17),
                                      (3, 2, 33), (2, 3, 65), (1, 2, 5)])
def test_2d_degenerate_lattices(nx, ny, nv):
    """Lattices of one or a few sites per axis (every streaming shift wraps
    several times; all but a few lanes of a workgroup are duplicates),
    velocity stride 4 and two collision sub-steps."""
    say(f"2d degenerate {nx}x{ny} nv={nv}")
    f0, u, p = make_case(2, nx, nv, ny=ny, seed=600 + 7 * nx + ny + nv,
                         slices=2, s=4, nsub=2)
    got = run_gpu(f0, u, p, 4, u_hold=2)
    want = run_oracle(f0, u, p, 4, u_hold=2)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2


@pytest.mark.parametrize("nv", [3, 5, 9, 17, 33])
def test_2d_f64_parity(nv):
    say(f"2d f64 nv={nv}")
    f0, u, p = make_case(2, 40, nv, ny=6, seed=500 + nv, dtype="f64")
    got = run_gpu(f0, u, p, 3, dtype="f64")
    want = run_oracle(f0, u, p, 3)
    assert rel_l2(got, want) <= FP64_REL_L2


@pytest.mark.parametrize("dim", [1, 2])
def test_nsub_stride_and_u_hold(dim):
    """nsub = 3 collision sub-steps, velocity stride 4 (coarse lattice),
    three u slices held two steps each."""
    say(f"nsub/stride/u_hold dim={dim}")
    nv = 9
    if dim == 1:
        f0, u, p = make_case(1, 130, nv, seed=7, slices=3, s=4, nsub=3)
    else:
        f0, u, p = make_case(2, 50, nv, ny=11, seed=8, slices=3, s=4, nsub=3)
    got = run_gpu(f0, u, p, 6, u_hold=2)
    want = run_oracle(f0, u, p, 6, u_hold=2)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2


@pytest.mark.parametrize("dim", [1, 2])
def test_drift_without_diffusion(dim):
    """kappa = 0 is accepted and gives the oracle's drift-only update."""
    nx, ny = (300, 1) if dim == 1 else (70, 5)
    say(f"{dim}d drift only (kappa = 0)")
    f0, u, p = make_case(dim, nx, 17, ny=ny, seed=920 + dim)
    p = dict(p, kappa=0.0)
    got = run_gpu(f0, u, p, 4)
    want = run_oracle(f0, u, p, 4)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2


def test_work_runs_on_the_given_stream():
    """The library queues its work on the stream it is given: a side stream
    is held up by a bounded GPU sleep, then the state is refilled and
    stepped on it with no host synchronisation in between; work queued
    anywhere else would read the zeros left before the refill."""
    import torch
    from paper_1508_02899_amd import Lattice
    from helpers import spec_for
    say("2d step queued behind a sleeping side stream")
    f0, u, p = make_case(2, 70, 9, ny=6, seed=930)
    want = run_oracle(f0, u, p, 3)
    side = torch.cuda.Stream()  # default priority
    lat = Lattice(spec_for(f0, p, "f32"), stream=side)
    src = torch.from_numpy(np.ascontiguousarray(f0)).cuda()
    ut = torch.from_numpy(np.ascontiguousarray(u)).cuda()
    f = torch.zeros_like(src)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.cuda._sleep(50_000_000)  # about 20 ms of spinning
        f.copy_(src)
    lat.step(f, ut, p["tau_p"], p["kappa"], p["dt"], 3)
    lat.sync()
    torch.cuda.synchronize()
    err = rel_l2(f.cpu().numpy(), want)
    lat.close()
    say("  rel L2", err)
    assert err <= FP32_REL_L2


@pytest.mark.parametrize("dim,nv", [(1, 33), (1, 129), (2, 9), (2, 33)])
def test_pure_streaming_bit_exact(dim, nv):
    """tau_p = inf and kappa = 0: exact periodic permutation (np.roll)."""
    say(f"streaming dim={dim} nv={nv}")
    if dim == 1:
        f0, u, p = make_case(1, 200, nv, seed=9)
    else:
        f0, u, p = make_case(2, 33, nv, ny=10, seed=10)
    p = dict(p, tau_p=math.inf, kappa=0.0)
    nsteps = 5
    got = run_gpu(f0, u, p, nsteps)
    h = (nv - 1) // 2
    if dim == 1:
        want = np.stack([np.roll(f0[j], (j - h) * nsteps) for j in range(nv)])
    else:
        want = np.empty_like(f0)
        for jy in range(nv):
            for jx in range(nv):
                want[jy * nv + jx] = np.roll(
                    f0[jy * nv + jx], ((jy - h) * nsteps, (jx - h) * nsteps),
                    axis=(0, 1))
    assert np.array_equal(got, want)


@pytest.mark.parametrize("dim", [1, 2])
def test_translation_and_determinism_bit_exact(dim):
    """Rolling f and u by (3, 5) sites rolls the GPU result exactly, and two
    runs are bit-identical (tile placement does not change arithmetic)."""
    nv = 33 if dim == 1 else 17
    if dim == 1:
        f0, u, p = make_case(1, 600, nv, seed=11)
        sh, ax, axu = 5, (1,), (2,)
        shift = (sh,)
    else:
        f0, u, p = make_case(2, 96, nv, ny=8, seed=12)
        shift, ax, axu = (3, 5), (1, 2), (2, 3)
    a = run_gpu(f0, u, p, 5)
    b = run_gpu(f0, u, p, 5)
    assert np.array_equal(a, b)
    c = run_gpu(np.ascontiguousarray(np.roll(f0, shift, axis=ax)),
                np.ascontiguousarray(np.roll(u, shift, axis=axu)), p, 5)
    assert np.array_equal(np.roll(a, shift, axis=ax), c)


@pytest.mark.parametrize("dim,dtype", [(1, "f64"), (2, "f64"), (1, "f32"),
                                       (2, "f32")])
def test_moments_and_mass_conservation(dim, dtype):
    """FP64 moments on the GPU equal the oracle's moments of the same state;
    mass is conserved to 1e-12 (FP64 state) / 1e-6 (FP32 state)."""
    import torch
    import oracle
    from paper_1508_02899_amd import Lattice
    from helpers import spec_for
    if dim == 1:
        f0, u, p = make_case(1, 512, 33, seed=13, dtype=dtype)
    else:
        f0, u, p = make_case(2, 64, 17, ny=16, seed=14, dtype=dtype)
    lat = Lattice(spec_for(f0, p, dtype))
    f = torch.from_numpy(f0).cuda()
    ut = torch.from_numpy(u).cuda()
    m0 = lat.moments(f, p["dt"])
    o0 = oracle.moments(f0, dim=dim, dx=p["dx"], dt=p["dt"])
    assert m0["mass"] == pytest.approx(o0["mass"], rel=1e-13)
    for k in range(dim):
        assert m0["momentum"][k] == pytest.approx(o0["momentum"][k], rel=1e-11,
                                                  abs=1e-13)
        assert m0["second_moment"][k] == pytest.approx(o0["second_moment"][k],
                                                       rel=1e-12)
    assert m0["variance"] == pytest.approx(o0["variance"], rel=1e-11)
    lat.step(f, ut, p["tau_p"], p["kappa"], p["dt"], 40)
    m1 = lat.moments(f, p["dt"])
    drift = abs(m1["mass"] - m0["mass"]) / m0["mass"]
    say(f"  mass drift {dtype} dim={dim}: {drift:.3e}")
    assert drift <= (1e-12 if dtype == "f64" else 1e-6)
    assert float(f.min()) >= -1e-7 * float(f.max())
    lat.close()


def test_density_matches_velocity_sum():
    import torch
    from paper_1508_02899_amd import Lattice
    from helpers import spec_for
    f0, u, p = make_case(2, 50, 9, ny=12, seed=15, dtype="f64")
    lat = Lattice(spec_for(f0, p, "f64"))
    rho = lat.density(torch.from_numpy(f0).cuda(), p["dt"]).cpu().numpy()
    dv = p["dx"] / p["dt"]
    np.testing.assert_allclose(rho, f0.sum(axis=0) * dv * dv, rtol=1e-14)
    lat.close()


def test_cfl_violation_is_sticky_and_leaves_f():
    """|u| past the bound of Eq. 3: flag set on the device, the call's
    steps are no-ops, lattice_sync reports ECFL once and clears it."""
    import torch
    from paper_1508_02899_amd import Lattice, LatticeError
    from paper_1508_02899_amd.lattice import ECFL
    from helpers import spec_for
    f0, u, p = make_case(1, 256, 17, seed=16)
    lat = Lattice(spec_for(f0, p, "f32"))
    f = torch.from_numpy(f0).cuda()
    bad = torch.from_numpy(u * 50.0).cuda()
    lat.step(f, bad, p["tau_p"], p["kappa"], p["dt"], 3)
    assert lat.sync(check=False) == ECFL
    assert np.array_equal(f.cpu().numpy(), f0)
    assert lat.sync(check=False) == 0  # cleared
    nan = torch.from_numpy(u).cuda()
    nan[0, 0, 5] = float("nan")
    lat.step(f, nan, p["tau_p"], p["kappa"], p["dt"], 2)
    with pytest.raises(LatticeError):
        lat.sync()
    # a good call afterwards works
    lat.step(f, torch.from_numpy(u).cuda(), p["tau_p"], p["kappa"], p["dt"], 2)
    lat.sync()
    lat.close()


def test_host_side_errors():
    import torch
    from paper_1508_02899_amd import Lattice, LatticeError
    from paper_1508_02899_amd.lattice import EDIFF, EINVAL, ECFL
    from helpers import spec_for
    f0, u, p = make_case(1, 64, 9, seed=17)
    lat = Lattice(spec_for(f0, p, "f32"))
    f = torch.from_numpy(f0).cuda()
    ut = torch.from_numpy(u).cuda()
    dv = p["dx"] / p["dt"]
    with pytest.raises(LatticeError) as e:
        lat.step(f, ut, p["tau_p"], 0.6 * dv * dv / p["dt"], p["dt"], 1)
    assert e.value.code == EDIFF
    with pytest.raises(LatticeError) as e:
        lat.step(f, ut, -1.0, p["kappa"], p["dt"], 1)
    assert e.value.code == EINVAL
    with pytest.raises(LatticeError) as e:  # Vmax alone violates CFL
        lat.step(f, ut, 1e-6, p["kappa"], p["dt"], 1)
    assert e.value.code == ECFL
    with pytest.raises(LatticeError) as e:  # not enough u slices
        from paper_1508_02899_amd import LatticeSpec
        lat2 = Lattice(LatticeSpec(dim=1, nx=64, nv=9, dx=p["dx"], u_hold=1))
        lat2.step(f, ut, p["tau_p"], p["kappa"], p["dt"], 3)
    assert e.value.code == EINVAL
    lat.step(f, ut, p["tau_p"], p["kappa"], p["dt"], 0)  # no-op
    assert np.array_equal(f.cpu().numpy(), f0)
    lat.close()


@pytest.mark.parametrize("padded", [True, False])
def test_2d_512x512_v33_full_size_sampled_sites(padded):
    """2D 512^2 x 33^2 FP32 (1.14 GB state), the bench launch (padded
    planes at the recommended pitch, as the benchmark runs) and the
    contiguous layout: one step on the GPU; 64 sampled sites (corners,
    edges, interior) recomputed one by one by the oracle from their
    streamed velocity columns."""
    import torch
    import oracle
    from paper_1508_02899_amd import Lattice, LatticeSpec, inputs
    from paper_1508_02899_amd.lattice import recommended_pitch
    say(f"config-3 full size sampled parity, padded={padded}")
    n, nv, L = 512, 33, 2 * math.pi
    h = (nv - 1) // 2
    u = inputs.flow2d_streamfunction(n, L, 1, seed=inputs.seed_for(3))
    vmax = 3.0
    dv = vmax / h
    dx = L / n
    dt = dx / dv
    tau_p = 2 * math.pi  # St = 1
    p = dict(dim=2, dx=dx, dt=dt, tau_p=tau_p, kappa=1e-4, s=1, nsub=1,
             scheme="koren")
    rng = np.random.default_rng(16)
    f0 = torch.rand((nv * nv, n, n), generator=torch.Generator().manual_seed(3),
                    dtype=torch.float32)
    spec = LatticeSpec(dim=2, nx=n, ny=n, nv=nv, dx=dx)
    if padded:
        spec.plane_pitch = recommended_pitch(spec)
        assert spec.plane_pitch == n * n + 64
        fd = spec.state_from(f0)
    else:
        fd = f0.cuda()
    lat = Lattice(spec)
    lat.step(fd, torch.from_numpy(u).cuda(), tau_p, p["kappa"], dt, 1)
    lat.sync()
    out = fd.cpu().numpy()
    f0n = f0.numpy()
    sites = [(0, 0), (0, n - 1), (n - 1, 0), (n - 1, n - 1), (5, 17), (511, 200)]
    sites += [tuple(rng.integers(0, n, 2)) for _ in range(58)]
    jy, jx = np.divmod(np.arange(nv * nv), nv)
    worst = 0.0
    for (y, x) in sites:
        col = f0n[np.arange(nv * nv), (y - (jy - h)) % n, (x - (jx - h)) % n]
        uu = u[:, :, y:y + 1, x:x + 1].astype(np.float64)
        # a 1x1 periodic lattice: streaming is the identity, the oracle
        # applies exactly the collision of this site
        ref = oracle.step(col.reshape(nv * nv, 1, 1).astype(np.float64), uu,
                          dim=2, dx=dx, tau_p=tau_p, kappa=p["kappa"], dt=dt,
                          nsteps=1)
        worst = max(worst, rel_l2(out[:, y, x], ref[:, 0, 0]))
    say("  worst site rel L2", worst)
    assert worst <= FP32_REL_L2
    lat.close()


def test_1d_16384x129_full_size_full_state():
    """1D 16384 x 129 FP32 (configuration 2 shape: 32 OU modes with k^-5/3
    variance, St = 1, Vmax = 2, kappa = 1e-4, one flow slice per step,
    Koren), 6 steps on the GPU against the oracle over the whole state."""
    import torch
    from paper_1508_02899_amd import Lattice, LatticeSpec, inputs
    say("config-2 full size parity")
    n, nv, L, steps = 16384, 129, 2 * math.pi, 6
    h = (nv - 1) // 2
    dx = L / n
    dv = 2.0 / h
    dt = dx / dv
    tau_p = 2 * math.pi
    u = inputs.flow1d(n, L, steps, modes=32, spectrum="k-5/3", tau_f=1.0,
                      dt=dt, seed=inputs.seed_for(2))
    f0 = inputs.gaussian_ic(1, n, nv, dx, dv)
    p = dict(dim=1, dx=dx, dt=dt, tau_p=tau_p, kappa=1e-4, s=1, nsub=1,
             scheme="koren", u_hold=1)
    lat = Lattice(LatticeSpec(dim=1, nx=n, nv=nv, dx=dx, u_hold=1))
    fd = torch.from_numpy(f0).cuda()
    lat.step(fd, torch.from_numpy(u).cuda(), tau_p, p["kappa"], dt, steps)
    lat.sync()
    got = fd.cpu().numpy()
    want = run_oracle(f0, u, p, steps, u_hold=1)
    err = rel_l2(got, want)
    say("  rel L2", err)
    assert err <= FP32_REL_L2
    lat.close()


def test_2d_256x256_v65_full_size_sampled_sites():
    """2D 256^2 x 65^2 FP32 (the fine lattice of configuration 5, 1.1 GB
    state), St = 2 with 4 collision sub-steps: one step on the GPU; 40
    sampled sites recomputed one by one by the oracle."""
    import torch
    import oracle
    from paper_1508_02899_amd import Lattice, LatticeSpec, inputs
    say("config-5 fine lattice full size sampled parity")
    n, nv, L, nsub = 256, 65, 2 * math.pi, 4
    h = (nv - 1) // 2
    u = inputs.flow2d_streamfunction(n, L, 1, seed=inputs.seed_for(5))
    dv = 3.0 / h
    dx = L / n
    dt = dx / dv
    tau_p = 2 * 2 * math.pi  # St = 2
    kappa = 1e-4
    f0 = torch.rand((nv * nv, n, n), generator=torch.Generator().manual_seed(5),
                    dtype=torch.float32)
    lat = Lattice(LatticeSpec(dim=2, nx=n, ny=n, nv=nv, dx=dx, nsub=nsub))
    ud = torch.from_numpy(u).cuda()
    cfl, _ = lat.stability(ud, tau_p, kappa, dt)
    assert cfl <= 0.5
    fd = f0.cuda()
    lat.step(fd, ud, tau_p, kappa, dt, 1)
    lat.sync()
    out = fd.cpu().numpy()
    f0n = f0.numpy()
    rng = np.random.default_rng(17)
    sites = [(0, 0), (n - 1, n - 1), (0, n - 1), (128, 3)]
    sites += [tuple(rng.integers(0, n, 2)) for _ in range(36)]
    jy, jx = np.divmod(np.arange(nv * nv), nv)
    worst = 0.0
    for (y, x) in sites:
        col = f0n[np.arange(nv * nv), (y - (jy - h)) % n, (x - (jx - h)) % n]
        uu = u[:, :, y:y + 1, x:x + 1].astype(np.float64)
        ref = oracle.step(col.reshape(nv * nv, 1, 1).astype(np.float64), uu,
                          dim=2, dx=dx, tau_p=tau_p, kappa=kappa, dt=dt,
                          nsteps=1, nsub=nsub)
        worst = max(worst, rel_l2(out[:, y, x], ref[:, 0, 0]))
    say("  worst site rel L2", worst)
    assert worst <= FP32_REL_L2
    lat.close()


@pytest.mark.parametrize("nx,nv,dtype,s,nsub,hold,nsteps,scheme", [
    (1, 3, "f32", 1, 1, 0, 5, "koren"),       # sites repeat in the region
    (31, 5, "f64", 1, 1, 1, 17, "koren"),
    (33, 7, "f32", 3, 1, 2, 19, "upwind"),
    (64, 9, "f64", 1, 2, 3, 40, "koren"),
    (200, 13, "f32", 2, 1, 1, 11, "koren"),
    (97, 17, "f64", 1, 1, 1, 9, "upwind"),
    (257, 17, "f32", 4, 3, 0, 7, "koren"),    # two steps per launch
    (256, 17, "f32", 8, 1, 0, 4, "koren"),    # the halo leaves no room
    (1000, 21, "f32", 1, 1, 4, 13, "koren"),
    (130, 25, "f64", 1, 5, 1, 6, "koren"),
    (256, 33, "f64", 1, 1, 1, 23, "koren"),
    (256, 33, "f32", 2, 1, 0, 6, "upwind"),
    (8192, 33, "f32", 1, 1, 1, 5, "koren"),   # 32-site tiles up to here
    (8193, 33, "f32", 1, 1, 1, 5, "koren"),   # 64-site tiles from here
    (8257, 17, "f64", 1, 2, 2, 9, "koren"),
    (16385, 9, "f64", 1, 1, 1, 6, "koren")])
def test_1d_several_steps_per_launch(nx, nv, dtype, s, nsub, hold, nsteps,
                                     scheme):
    """Short lattices take several steps per launch: a call of nsteps steps
    against the oracle, against calls of one step (the same bits where the
    one-step pass is the split-column one, nv 17 and 33), and a call whose
    flow breaks the CFL bound in its last slice leaves f alone."""
    import torch
    from helpers import spec_for
    from paper_1508_02899_amd import Lattice, LatticeError
    slices = -(-nsteps // hold) if hold else 1
    f0, u, p = make_case(1, nx, nv, dtype=dtype, seed=nx + nv, slices=slices,
                         s=s, nsub=nsub, scheme=scheme)
    spec = spec_for(f0, p, dtype, hold)
    ud = torch.from_numpy(u).cuda()
    args = (p["tau_p"], p["kappa"], p["dt"])
    with Lattice(spec) as lat:
        fa = torch.from_numpy(f0).cuda()
        lat.step(fa, ud, *args, nsteps)
        lat.sync()
        fb = torch.from_numpy(f0).cuda()
        for n in range(nsteps):
            k = n // hold if hold else 0
            lat.step(fb, ud[k:k + 1].contiguous(), *args, 1)
        lat.sync()
        fc = torch.from_numpy(f0).cuda()
        bad = ud.clone()
        bad[-1, 0, nx // 2] = float("nan")
        lat.step(fc, bad, *args, nsteps)
        with pytest.raises(LatticeError):
            lat.sync()
        assert torch.equal(fc, torch.from_numpy(f0).cuda())
    bound = FP32_REL_L2 if dtype == "f32" else FP64_REL_L2
    err = rel_l2(fa.cpu().numpy(), run_oracle(f0, u, p, nsteps, u_hold=hold))
    say(f"  rel L2 {err:.2e}")
    assert err <= bound
    if nv in (17, 33):
        assert torch.equal(fa, fb)
    else:
        assert rel_l2(fa.cpu().numpy(), fb.cpu().numpy()) <= bound


@pytest.mark.parametrize("nv,dtype,nx,ny,scheme", [
    (7, "f32", 33, 7, "koren"), (9, "f32", 70, 5, "upwind"),
    (9, "f32", 1101, 16, "koren"), (11, "f32", 65, 3, "koren"),
    (13, "f32", 17, 9, "koren"), (15, "f32", 40, 6, "upwind"),
    (17, "f32", 9, 8, "koren"), (17, "f32", 137, 67, "koren"),
    (17, "f32", 137, 270, "koren"), (19, "f32", 33, 5, "koren"),
    (21, "f32", 50, 4, "upwind"), (25, "f32", 13, 5, "koren"),
    (33, "f32", 5, 3, "koren"), (33, "f32", 67, 70, "upwind"),
    (33, "f32", 132, 67, "koren"), (65, "f32", 7, 5, "koren"),
    (9, "f64", 35, 6, "koren"), (17, "f64", 21, 5, "koren"),
    (33, "f64", 6, 5, "koren"), (33, "f64", 40, 66, "koren")])
def test_2d_small_lattice_shapes(nv, dtype, nx, ny, scheme):
    """Every shape of the small-lattice pass (4, 2 and 1 times the parts, one
    wavefront per workgroup) with ragged tiles: against the oracle, and the
    same bits as the pass of a lattice too large for it (the same sites
    repeated along y, which the update does not notice)."""
    import torch
    from paper_1508_02899_amd import Lattice
    from helpers import spec_for
    f0, u, p = make_case(2, nx, nv, ny=ny, dtype=dtype, seed=nx * ny + nv,
                         scheme=scheme)
    bound = FP32_REL_L2 if dtype == "f32" else FP64_REL_L2
    got = run_gpu(f0, u, p, 2, dtype)
    err = rel_l2(got, run_oracle(f0, u, p, 2))
    say(f"  rel L2 {err:.2e}")
    assert err <= bound
    reps = 2600 * 64 // (nx * ny) + 1  # past 2600 wavefronts at any shape
    if reps * f0.nbytes <= 2 << 30:
        fb = np.tile(f0, (1, reps, 1))
        ub = np.tile(u, (1, 1, reps, 1))
        q = dict(p)
        with Lattice(spec_for(fb, q, dtype)) as lat:
            fd = torch.from_numpy(fb).cuda()
            lat.step(fd, torch.from_numpy(ub).cuda(), p["tau_p"], p["kappa"],
                     p["dt"], 2)
            lat.sync()
            assert np.array_equal(fd[:, :ny].cpu().numpy(), got)


@pytest.mark.parametrize("nv,dtype,nx,ny,scheme", [
    (5, "f32", 70, 9, "koren"), (5, "f64", 33, 4, "upwind"),
    (9, "f32", 37, 5, "upwind"), (9, "f64", 19, 6, "koren"),
    (13, "f32", 50, 7, "koren"), (17, "f32", 130, 11, "koren"),
    (17, "f64", 9, 5, "koren"), (21, "f32", 33, 8, "koren"),
    (25, "f32", 12, 6, "upwind"), (33, "f32", 17, 9, "koren"),
    (33, "f64", 6, 5, "koren"), (65, "f32", 6, 5, "koren"),
    # the shapes of states past 128 MB, and a lattice of one pass per sub-step
    (65, "f32", 97, 83, "koren"), (33, "f32", 203, 160, "upwind"),
    (25, "f32", 301, 181, "koren"), (17, "f32", 350, 339, "koren"),
    (17, "f64", 64, 70, "koren"), (7, "f32", 40, 9, "koren")])
def test_2d_sub_steps_in_one_pass(nv, dtype, nx, ny, scheme):
    """2, 3, 4 and 5 collision sub-steps (one to three passes): bit for bit
    the streaming followed by single collisions with the same coefficients
    (2 and 4: tau_p and kappa scale by powers of two), the small ones also
    against the oracle."""
    import torch
    from dataclasses import replace
    from helpers import spec_for
    from paper_1508_02899_amd import Lattice
    bound = FP32_REL_L2 if dtype == "f32" else FP64_REL_L2
    small = nx * ny * nv * nv < 1 << 20
    for nsub in (2, 3, 4, 5):
        f0, u, p = make_case(2, nx, nv, ny=ny, dtype=dtype, seed=nv + nsub,
                             nsub=nsub, scheme=scheme)
        spec = spec_for(f0, p, dtype)
        ud = torch.from_numpy(u).cuda()
        f = torch.from_numpy(f0).cuda()
        with Lattice(spec) as lat:
            lat.step(f, ud, p["tau_p"], p["kappa"], p["dt"], 1)
            lat.sync()
        if small:
            err = rel_l2(f.cpu().numpy(), run_oracle(f0, u, p, 1))
            say(f"  nsub {nsub}: rel L2 {err:.2e}")
            assert err <= bound
        if nsub in (2, 4):
            g = torch.from_numpy(f0).cuda()
            with Lattice(replace(spec, nsub=1)) as one:
                one.step(g, ud, math.inf, 0.0, p["dt"], 1)
                for _ in range(nsub):
                    one.collide(g, ud, nsub * p["tau_p"], p["kappa"] / nsub,
                                p["dt"], 1)
                one.sync()
            assert torch.equal(f, g)


def test_2d_sub_steps_cfl_violation_leaves_f():
    import torch
    from helpers import spec_for
    from paper_1508_02899_amd import Lattice, LatticeError
    f0, u, p = make_case(2, 40, 17, ny=9, seed=5, nsub=3)
    u[0, 1, 4, 7] = np.inf
    f = torch.from_numpy(f0).cuda()
    with Lattice(spec_for(f0, p, "f32")) as lat:
        lat.step(f, torch.from_numpy(u).cuda(), p["tau_p"], p["kappa"],
                 p["dt"], 2)
        with pytest.raises(LatticeError):
            lat.sync()
    assert np.array_equal(f.cpu().numpy(), f0)


@pytest.mark.parametrize("nv,nx,ny", [(5, 350, 401), (9, 203, 160),
                                      (17, 150, 131), (33, 70, 45)])
def test_2d_fp64_upwind_sub_steps_of_many_sites(nv, nx, ny):
    """FP64 upwind lattices past 2500 wavefronts, whose sub-steps share a
    pass there too."""
    test_2d_sub_steps_in_one_pass(nv, "f64", nx, ny, "upwind")


@pytest.mark.parametrize("nx,nsub,scheme", [(301, 1, "koren"),
                                            (97, 3, "upwind")])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nv", [3, 5, 7, 9, 11, 13, 17, 21, 25, 33, 45, 65])
def test_1d_bits_do_not_depend_on_the_call(nv, dtype, nx, nsub, scheme):
    """The same bits from one call of n steps, n calls of one step, a call
    with profiling on, a state that is not 16-byte aligned and the step that
    allocates nothing: several passes serve them, with one arithmetic."""
    import torch
    from helpers import spec_for
    from paper_1508_02899_amd import Lattice
    from paper_1508_02899_amd.lattice import step_noalloc
    f0, u, p = make_case(1, nx, nv, dtype=dtype, seed=nx + nv, nsub=nsub,
                         scheme=scheme)
    spec = spec_for(f0, p, dtype)
    start, ud = torch.from_numpy(f0).cuda(), torch.from_numpy(u).cuda()
    args = (p["tau_p"], p["kappa"], p["dt"])
    with Lattice(spec) as lat:
        def call(nsteps, off=0):
            buf = torch.empty(start.numel() + off, dtype=start.dtype,
                              device="cuda")
            f = buf[off:].view(start.shape)
            f.copy_(start)
            lat.step(f, ud, *args, nsteps)
            lat.sync()
            return f
        ref = start.clone()
        for n in range(1, 8):
            lat.step(ref, ud, *args, 1)
            lat.sync()
            for off in (0, 1):
                assert torch.equal(call(n, off), ref), f"{n} steps, {off}"
        lat.profile(True)
        assert torch.equal(call(7), ref)
        lat.profile(False)
    f = start.clone()
    step_noalloc(spec, f, ud, *args, 7)
    assert torch.equal(f, ref)


@pytest.mark.parametrize("nv,dtype,nx,ny,scheme,cut", [
    (5, "f32", 161, 205, "koren", True), (9, "f32", 211, 130, "upwind", True),
    (17, "f32", 203, 90, "koren", True), (33, "f32", 111, 104, "koren", True),
    (65, "f32", 101, 79, "koren", True), (25, "f32", 305, 200, "koren", True),
    (17, "f64", 131, 90, "upwind", True), (9, "f64", 60, 30, "koren", False),
    (17, "f32", 40, 30, "koren", False), (33, "f32", 177, 132, "koren", False)])
def test_2d_odd_number_of_passes(nv, dtype, nx, ny, scheme, cut):
    """Calls of one and three steps whose sub-steps share passes: a large
    state is never copied (an even number of passes, the first one in two
    halves), a small one may be; the bits are those of the streaming followed
    by single collisions either way, also from the step that allocates
    nothing."""
    import torch
    from dataclasses import replace
    from helpers import spec_for
    from paper_1508_02899_amd import Lattice
    from paper_1508_02899_amd.lattice import NOALLOC_MAX_BYTES, step_noalloc
    for nsub, nsteps in ((2, 1), (2, 3), (4, 1)):
        f0, u, p = make_case(2, nx, nv, ny=ny, dtype=dtype, seed=nv + nsub,
                             nsub=nsub, scheme=scheme)
        spec = spec_for(f0, p, dtype)
        start, ud = torch.from_numpy(f0).cuda(), torch.from_numpy(u).cuda()
        args = (p["tau_p"], p["kappa"], p["dt"])
        f = start.clone()
        with Lattice(spec) as lat:
            lat.profile(True)
            lat.step(f, ud, *args, nsteps)
            lat.sync()
            passes = lat.profile_read()[1]
        say(f"  nsub {nsub}, {nsteps} steps: {passes} passes")
        if cut:
            assert passes % 2 == 0
        elif nsub == 2:
            assert passes == nsteps
        g = start.clone()
        with Lattice(replace(spec, nsub=1)) as one:
            for _ in range(nsteps):
                one.step(g, ud, math.inf, 0.0, p["dt"], 1)
                for _ in range(nsub):
                    one.collide(g, ud, nsub * p["tau_p"], p["kappa"] / nsub,
                                p["dt"], 1)
            one.sync()
        assert torch.equal(f, g)
        if f0.nbytes <= NOALLOC_MAX_BYTES:
            g = start.clone()
            step_noalloc(spec, g, ud, *args, nsteps)
            assert torch.equal(f, g)
        del f, g, start


@pytest.mark.parametrize("nv,nx,ny,scheme,nsub,passes", [
    (21, 228, 174, "koren", 3, 3), (21, 160, 114, "koren", 2, 2),
    (21, 228, 174, "upwind", 3, 1), (21, 128, 93, "koren", 3, 1),
    (17, 272, 199, "koren", 2, 2), (17, 240, 182, "koren", 2, 1),
    (25, 192, 135, "koren", 4, 4), (5, 1984, 1519, "koren", 2, 2),
    (5, 1408, 1074, "koren", 2, 1), (9, 1104, 843, "koren", 2, 1)])
def test_2d_sub_steps_share_a_pass_only_where_it_is_shorter(nv, nx, ny, scheme,
                                                           nsub, passes):
    """Passes of a step on lattices where a pass per sub-step is the faster
    form (Koren: 21^2 from 800 wavefronts, others from 3000, 5^2 past 256
    MB), and on their neighbours where it is not."""
    import torch
    from paper_1508_02899_amd import Lattice, LatticeSpec
    spec = LatticeSpec(dim=2, nx=nx, ny=ny, nv=nv, dx=0.1, scheme=scheme,
                       nsub=nsub)
    dv = 3.0 / ((nv - 1) // 2)
    dt = 0.1 / dv
    f = torch.ones(spec.state_shape, device="cuda")
    u = torch.zeros(spec.u_shape(1), device="cuda")
    with Lattice(spec) as lat:
        lat.profile(True)
        lat.step(f, u, dt / (nsub * dv) * 15, 1e-6, dt, 2)
        lat.sync()
        assert lat.profile_read()[1] == 2 * passes


@pytest.mark.parametrize("nv,dtype,nx,ny", [
    (33, "f32", 109, 141), (33, "f32", 113, 141), (33, "f32", 150, 130),
    (65, "f32", 77, 65), (65, "f32", 77, 66), (33, "f64", 111, 55),
    (33, "f64", 111, 56)])
def test_2d_upwind_small_lattices_of_many_velocities(nv, dtype, nx, ny):
    """Both sides of the line at which upwind lattices of 33^2 and 65^2 go
    back to the default shape."""
    test_2d_small_lattice_shapes(nv, dtype, nx, ny, "upwind")


@pytest.mark.parametrize("nx,nv,dtype,nsub,nsteps", [
    # both sides of every line of the rule (sites by weight of the update),
    # with step counts that need an odd number of launches, spread unevenly
    (65536, 9, "f32", 1, 33), (65537, 9, "f32", 1, 5),
    (32768, 33, "f32", 1, 9), (32768, 17, "f64", 1, 19),
    (32769, 17, "f64", 1, 3), (32768, 13, "f32", 3, 23),
    (32769, 13, "f32", 3, 3), (16384, 5, "f32", 8, 33),
    (16385, 5, "f32", 8, 3), (8192, 5, "f64", 5, 33), (8193, 5, "f64", 5, 3),
    (200, 9, "f64", 6, 3), (8192, 33, "f64", 1, 9)])
def test_1d_several_steps_at_the_ends_of_their_ranges(nx, nv, dtype, nsub,
                                                      nsteps):
    """Aligned and with the state one element off: the bits of single steps,
    and the oracle's values."""
    import torch
    from helpers import spec_for
    from paper_1508_02899_amd import Lattice
    f0, u, p = make_case(1, nx, nv, dtype=dtype, seed=nx + nv, nsub=nsub)
    spec = spec_for(f0, p, dtype)
    start, ud = torch.from_numpy(f0).cuda(), torch.from_numpy(u).cuda()
    args = (p["tau_p"], p["kappa"], p["dt"])
    with Lattice(spec) as lat:
        ref = start.clone()
        for _ in range(nsteps):
            lat.step(ref, ud, *args, 1)
        lat.sync()
        for off in (0, 1):
            buf = torch.full((start.numel() + off,), float("nan"),
                             dtype=start.dtype, device="cuda")
            f = buf[off:].view(start.shape)
            f.copy_(start)
            lat.step(f, ud, *args, nsteps)
            lat.sync()
            assert torch.equal(f, ref)
    bound = FP32_REL_L2 if dtype == "f32" else FP64_REL_L2
    err = rel_l2(ref.cpu().numpy(), run_oracle(f0, u, p, nsteps))
    say(f"  rel L2 {err:.2e}")
    assert err <= bound
