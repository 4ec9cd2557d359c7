"""GPU S1(r) (Eq. 11) vs the FP64 oracle (oracle/structure.py)."""
import math

import numpy as np
import pytest

from helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,nx,ny,nv,dtype", [(1, 300, 1, 33, "f32"),
                                                (1, 128, 1, 65, "f64"),
                                                (2, 24, 16, 9, "f32"),
                                                (2, 20, 12, 17, "f64")])
def test_s1_matches_oracle(dim, nx, ny, nv, dtype):
    import torch
    from oracle import structure as S
    from paper_1508_02899_amd import Lattice, LatticeSpec
    rng = np.random.default_rng(80 + nx)
    shape = (nv, nx) if dim == 1 else (nv * nv, ny, nx)
    f = rng.random(shape) ** 3
    f = f.astype(np.float32 if dtype == "f32" else np.float64)
    dx, dt = 2 * math.pi / nx, 0.07
    lat = Lattice(LatticeSpec(dim=dim, nx=nx, ny=ny, nv=nv, dx=dx,
                              dtype=dtype))
    rs = [0, 1, 2, 5, 11, nx - 1]
    got = lat.s1(torch.from_numpy(f).cuda(), dt, rs)
    want = S.s1(f, dim, dx / dt, rs)
    err = np.max(np.abs(got - want) / np.abs(want))
    say(f"  S1 {np.round(got[:4], 5)}; max rel err {err:.2e}")
    assert err < (1e-5 if dtype == "f32" else 1e-12)
    lat.close()


@pytest.mark.parametrize("dim,nx,ny,nv,dtype,pad,nr", [
    (1, 1, 1, 3, "f32", 0, 1), (1, 511, 1, 9, "f32", 0, 4),
    (1, 513, 1, 17, "f64", 0, 5), (2, 33, 31, 9, "f32", 7, 2),
    (2, 40, 37, 5, "f64", 0, 6), (2, 31, 17, 9, "f32", 0, 8),
    (2, 24, 16, 9, "f32", 0, 9), (2, 16, 9, 5, "f32", 0, 33)])
def test_s1_sets_of_separations(dim, nx, ny, nv, dtype, pad, nr):
    """Every set size (4, 8, 12, 16 separations at once, several sets, a
    workspace that grows), chunks of sites with a remainder, separations
    past the lattice, a padded pitch; and steps around the call come out as
    without it (the call uses the handle's scratch).  Tolerances as in the
    test above: FP32 h within 1e-5, FP64 within 1e-12."""
    import torch
    from oracle import structure as S
    from paper_1508_02899_amd import Lattice, LatticeSpec
    rng = np.random.default_rng(90 + nx + nr)
    shape = (nv, nx) if dim == 1 else (nv * nv, ny, nx)
    f = rng.random(shape) ** 3 + 0.01
    f = f.astype(np.float32 if dtype == "f32" else np.float64)
    dx, dt = 2 * math.pi / nx, 0.07
    spec = LatticeSpec(dim=dim, nx=nx, ny=ny, nv=nv, dx=dx, dtype=dtype,
                       plane_pitch=nx * ny + pad if pad else 0)
    rs = [int(r) for r in rng.integers(0, 3 * max(nx, ny), nr)]
    rs[0] = 0
    u = torch.zeros(spec.u_shape(1), device="cuda",
                    dtype=torch.float32 if dtype == "f32" else torch.float64)
    states = []
    for probe in (False, True):
        with Lattice(spec) as lat:
            fd = spec.state_from(f)
            if probe:
                lat.s1(fd, dt, rs[:1])
                got = lat.s1(fd, dt, rs)
                assert np.array_equal(got, lat.s1(fd, dt, rs))
            for n in (1, 2):
                lat.step(fd, u, math.inf, 0.0, dt, n)
                if probe:
                    lat.s1(fd, dt, rs[:1])
            states.append(fd.cpu().numpy())
    assert np.array_equal(states[0], states[1])
    want = S.s1(f, dim, dx / dt, [r % nx for r in rs]) if dim == 1 else \
        S.s1(f, dim, dx / dt, rs)
    err = np.max(np.abs(got - want) / np.abs(want))
    say(f"  max rel err {err:.2e}")
    assert err < (1e-5 if dtype == "f32" else 1e-12)


@pytest.mark.parametrize("dim,nx,ny,nv,dtype,pad,nr", [
    (1, 257, 1, 5, "f32", 0, 17), (1, 300, 1, 3, "f64", 0, 40),
    (1, 64, 1, 3, "f64", 0, 48), (1, 64, 1, 3, "f64", 0, 49),
    (1, 40, 1, 3, "f64", 0, 1000), (2, 17, 12, 3, "f64", 5, 70),
    (2, 12, 9, 3, "f32", 0, 600)])
def test_s1_many_sets_of_separations_in_a_launch(dim, nx, ny, nv, dtype, pad,
                                                 nr):
    """Several sets a launch, the last one not full, and several launches."""
    test_s1_sets_of_separations(dim, nx, ny, nv, dtype, pad, nr)
