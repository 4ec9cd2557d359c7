"""GPU <rho_r^2> on tilings vs the FP64 oracle (oracle/observables.py)."""
import math

import numpy as np
import pytest

from helpers import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,nx,ny,levels", [(2, 64, 32, 6), (2, 48, 16, 4),
                                              (1, 1024, 1, 11), (2, 8, 8, 1)])
def test_rho_r2_matches_oracle(dim, nx, ny, levels):
    import torch
    from oracle import observables as O
    from paper_1508_02899_amd import Lattice, LatticeSpec
    rng = np.random.default_rng(60 + nx)
    nv = 9
    shape = (nv ** dim, ny, nx) if dim == 2 else (nv, nx)
    f = (rng.random(shape) ** 4).astype(np.float32)
    dx = 2 * math.pi / nx
    dt = 0.1
    lat = Lattice(LatticeSpec(dim=dim, nx=nx, ny=ny, nv=nv, dx=dx))
    fd = torch.from_numpy(f).cuda()
    rho = lat.density(fd, dt)
    got = lat.rho_r2(rho, levels)
    dv = dx / dt
    want = O.rho_r2(O.density(f, dim, dv).reshape(ny, nx), levels)
    say(f"  <rho_r^2> {np.round(got, 4)}")
    assert np.allclose(got, want, rtol=1e-12, atol=0)
    # bit-reproducible
    assert np.array_equal(got, lat.rho_r2(rho, levels))
    lat.close()


@pytest.mark.parametrize("dim,nx,ny,levels", [
    (2, 31, 33, 1), (2, 34, 2, 2), (2, 96, 160, 6), (2, 64, 192, 7),
    (2, 128, 128, 8), (2, 2048, 1024, 11), (2, 1024, 3072, 7),
    (1, 1023, 1, 1), (1, 3 * 1024, 1, 11), (1, 4096, 1, 12),
    (1, 1 << 21, 1, 22), (1, 7 << 14, 1, 15)])
def test_rho_r2_stages_match_oracle(dim, nx, ny, levels):
    """Edge tiles, one and two stages, a last stage of one and of several
    workgroups.  Positive sums of n terms in any order agree within n 2^-53
    each (pairwise: far below 1e-12 here)."""
    import torch
    from oracle import observables as O
    from paper_1508_02899_amd import Lattice, LatticeSpec
    rng = np.random.default_rng(nx + ny)
    rho = rng.random((ny, nx)) ** 4 + 1e-3
    lat = Lattice(LatticeSpec(dim=dim, nx=nx, ny=ny, nv=3, dx=0.1))
    rd = torch.from_numpy(rho).cuda()
    got = lat.rho_r2(rd, levels)
    np.testing.assert_allclose(
        got, O.rho_r2(rho if dim == 2 else rho[0], levels), rtol=1e-12)
    assert np.array_equal(got[:1], lat.rho_r2(rd, 1))
    assert np.array_equal(got, lat.rho_r2(rd, levels))
    lat.close()


def test_rho_r2_rejects_bad_tiling():
    import torch
    from paper_1508_02899_amd import Lattice, LatticeSpec, LatticeError
    lat = Lattice(LatticeSpec(dim=2, nx=24, ny=16, nv=3, dx=0.1))
    rho = torch.ones((16, 24), dtype=torch.float64, device="cuda")
    assert lat.rho_r2(rho, 4)[0] == pytest.approx(1.0)
    with pytest.raises(LatticeError):
        lat.rho_r2(rho, 5)  # 24 is not a multiple of 16
    lat.close()


@pytest.mark.parametrize("dim,nx,ny,nv,dtype,pad", [
    (1, 1, 1, 3, "f32", 0), (1, 131, 1, 129, "f32", 0),
    (2, 37, 5, 9, "f64", 3), (2, 65, 3, 9, "f32", 1),
    (2, 63, 9, 33, "f32", 5),
    # 16-byte loads: from 131072 sites (FP32) and 65536 (FP64) on
    (1, 131072, 1, 33, "f32", 0), (1, 131076, 1, 65, "f32", 0),
    (2, 512, 256, 9, "f32", 64), (2, 512, 256, 9, "f32", 2),
    (1, 65538, 1, 65, "f64", 0), (1, 65539, 1, 17, "f64", 0)])
def test_density_sums_every_plane_once(dim, nx, ny, nv, dtype, pad):
    """Odd sizes, few and many planes, both load widths and pitches that
    rule the wide loads out, against a 64-bit sum of the same values; NaN in
    the padding must not be read.  Tolerance: n - 1 additions of positive
    terms and one product, each within 2^-53."""
    import torch
    from paper_1508_02899_amd import Lattice, LatticeSpec
    spec = LatticeSpec(dim=dim, nx=nx, ny=ny, nv=nv, dx=0.5, dtype=dtype,
                       plane_pitch=nx * ny + pad if pad else 0)
    lat = Lattice(spec)
    f = spec.empty_state()
    f.as_strided((spec.state_span,), (1,)).fill_(float("nan"))
    g = torch.Generator(device="cuda")
    g.manual_seed(nx + nv)
    f.copy_(torch.rand(f.shape, generator=g, device="cuda", dtype=f.dtype))
    dt = 0.25
    got = lat.density(f, dt)
    dv = 0.5 / dt
    want = f.double().sum(0).reshape(got.shape) * dv ** dim
    tol = (nv ** dim + 8) * 2.0 ** -53
    assert float(((got - want) / want).abs().max()) <= tol
    assert torch.equal(got, lat.density(f, dt))
    lat.close()


@pytest.mark.parametrize("dim,nx,ny,nv,dtype,pad", [
    # a lane per site where no wide load fits, two and eight loads in flight
    (1, 262143, 1, 17, "f32", 0), (1, 262145, 1, 17, "f32", 0),
    (1, 262145, 1, 129, "f32", 0), (2, 641, 411, 9, "f64", 0),
    (2, 641, 411, 11, "f32", 1),
    # planes 64 KiB apart: two wavefronts (FP32), a lane (FP64), and beside
    (1, 262144, 1, 17, "f32", 0), (2, 512, 512, 9, "f32", 0),
    (2, 512, 512, 9, "f32", 64), (1, 262144, 1, 9, "f32", 0),
    (2, 512, 512, 9, "f64", 0), (1, 262144, 1, 17, "f64", 0),
    (1, 524288, 1, 3, "f64", 0), (1, 1 << 21, 1, 3, "f64", 0),
    (1, (1 << 21) + 8192, 1, 3, "f64", 0)])
def test_density_of_many_sites(dim, nx, ny, nv, dtype, pad):
    """The forms for many sites on both sides of each line."""
    test_density_sums_every_plane_once(dim, nx, ny, nv, dtype, pad)
