"""Flow synthesis on the GPU from mode tables vs the FP64 oracle
(oracle/flows.py), and lattice steps driven by device-synthesised flows
vs the same steps with prestaged flows."""
import math

import numpy as np
import pytest

from helpers import rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,nx,K,ns", [("f32", 1000, 32, 7),
                                           ("f64", 256, 8, 3)])
def test_flow1d_modes_match_oracle(dtype, nx, K, ns):
    import torch
    from oracle import flows as F
    from paper_1508_02899_amd import Lattice, LatticeSpec, inputs
    tab = inputs.flow1d_modes(ns, modes=K, spectrum="k-5/3", tau_f=1.0,
                              dt=0.1, seed=21).astype(np.float32)
    lat = Lattice(LatticeSpec(dim=1, nx=nx, nv=9, dx=2 * math.pi / nx,
                              dtype=dtype))
    u = lat.flow_from_modes(torch.from_numpy(tab).cuda()).cpu().numpy()
    want = F.flow1d(tab, nx)
    err = rel_l2(u, want)
    say(f"  1D {dtype}: rel L2 {err:.2e}")
    assert err < (2e-6 if dtype == "f32" else 1e-12)
    lat.close()


@pytest.mark.parametrize("dtype,nx,ny,K,ns", [("f32", 96, 64, 16, 3),
                                              ("f32", 512, 512, 32, 1),
                                              ("f64", 40, 48, 8, 2)])
def test_flow2d_modes_match_oracle(dtype, nx, ny, K, ns):
    import torch
    from oracle import flows as F
    from paper_1508_02899_amd import Lattice, LatticeSpec
    rng = np.random.default_rng(22 + nx)
    tab = rng.standard_normal((ns, 2 * K + 1, K + 1, 2)).astype(np.float32)
    dx = 0.05
    lat = Lattice(LatticeSpec(dim=2, nx=nx, ny=ny, nv=3, dx=dx, dtype=dtype))
    u = lat.flow_from_modes(torch.from_numpy(tab).cuda()).cpu().numpy()
    want = F.flow2d(tab, nx, ny, dx)
    err = rel_l2(u, want)
    say(f"  2D {dtype} {nx}x{ny} K={K}: rel L2 {err:.2e}")
    assert err < (5e-6 if dtype == "f32" else 1e-12)
    lat.close()


@pytest.mark.parametrize("dtype,nx,ny,K,ns", [
    ("f32", 3, 3, 1, 1), ("f32", 131, 133, 64, 2), ("f64", 129, 131, 64, 1),
    ("f32", 65, 33, 15, 5), ("f64", 63, 31, 14, 3),
    ("f32", 2048, 130, 64, 17)])  # two chunks of slices
def test_flow2d_edges_and_chunks(dtype, nx, ny, K, ns):
    """Ragged tiles of sites and rows, the smallest and largest tables, more
    slices than the workspace holds at once, then a smaller call.  FP32: each
    of 2 K + 1 terms of a sum carries a few roundings of 2^-24, as in the
    test above."""
    import torch
    from oracle import flows as F
    from paper_1508_02899_amd import Lattice, LatticeSpec
    rng = np.random.default_rng(24 + nx)
    tab = rng.standard_normal((ns, 2 * K + 1, K + 1, 2)).astype(np.float32)
    lat = Lattice(LatticeSpec(dim=2, nx=nx, ny=ny, nv=3, dx=0.05,
                              dtype=dtype))
    td = torch.from_numpy(tab).cuda()
    u = lat.flow_from_modes(td).cpu().numpy()
    bound = 5e-6 if dtype == "f32" else 1e-12
    for s in sorted({0, ns // 2, ns - 1}):
        err = rel_l2(u[s], F.flow2d(tab[s:s + 1], nx, ny, 0.05)[0])
        assert err < bound, (s, err)
    v = lat.flow_from_modes(td[-1:].contiguous()).cpu().numpy()
    assert np.array_equal(u[-1:], v)
    lat.close()


def test_flow2d_under_capture():
    """A captured call replays on new tables after the handle's own
    workspace has grown."""
    import torch
    from paper_1508_02899_amd import Lattice, LatticeSpec
    st = torch.cuda.Stream()
    spec = LatticeSpec(dim=2, nx=64, ny=48, nv=3, dx=0.05)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    tabs = [torch.randn((2, 17, 9, 2), generator=g, device="cuda")
            for _ in range(3)]
    coef = tabs[0].clone()
    out = torch.empty((2, 2, 48, 64), device="cuda")
    lat = Lattice(spec, stream=st)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        lat.flow_from_modes(coef, out=out)
    big = torch.randn((9, 41, 21, 2), generator=g, device="cuda")
    for t in tabs:
        coef.copy_(t)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        lat.flow_from_modes(big)
        want = lat.flow_from_modes(t)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    lat.close()


@pytest.mark.parametrize("own_stream", [True, False])
@pytest.mark.parametrize("thread", [False, True])
def test_flow2d_while_another_stream_is_captured(thread, own_stream):
    """The first calls of a handle, the second with a larger workspace, while
    a graph is being captured on a stream that is not the handle's: both sides
    succeed (nothing that ends the capture is called)."""
    import threading

    import torch
    from paper_1508_02899_amd import Lattice, LatticeSpec
    spec = LatticeSpec(dim=2, nx=64, ny=48, nv=3, dx=0.05)
    st = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    tabs = [torch.randn((n, 2 * K + 1, K + 1, 2), device="cuda")
            for n, K in ((1, 4), (5, 20))]
    outs = [torch.empty((t.shape[0], 2, 48, 64), device="cuda") for t in tabs]
    x = torch.zeros(100, device="cuda")
    lat, errors = Lattice(spec, stream=st), []
    torch.cuda.synchronize()

    def calls():
        try:
            for t, o in zip(tabs, outs):
                lat.flow_from_modes(t, out=o)
        except Exception as e:  # reported by the test's own thread
            errors.append(e)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        x.add_(1)
        if thread:
            t = threading.Thread(target=calls)
            t.start()
            t.join()
        else:
            calls()
    assert not errors, errors
    graph.replay()
    torch.cuda.synchronize()
    assert bool((x == 1).all())
    again = [lat.flow_from_modes(t) for t in tabs]
    torch.cuda.synchronize()
    for o, a in zip(outs, again):
        assert torch.equal(o, a)
    lat.close()


def test_steps_with_device_flow_match_prestaged_flow():
    """2D Koren steps driven by flows synthesised on the device equal the
    steps driven by the prestaged inverse-FFT flows up to the FP32 rounding
    of u."""
    import torch
    from paper_1508_02899_amd import Lattice, LatticeSpec, inputs
    n, nv, L, steps = 64, 17, 2 * math.pi, 20
    dx = L / n
    dv = 3.0 / ((nv - 1) // 2)
    dt = dx / dv
    kw = dict(kmax=16, tau_f=1.0, dt=dt, seed=inputs.seed_for(3, 9))
    u_pre = torch.from_numpy(inputs.flow2d_streamfunction(n, L, steps, **kw)).cuda()
    tab = torch.from_numpy(inputs.flow2d_modes(n, L, steps, **kw)).cuda()
    spec = LatticeSpec(dim=2, nx=n, ny=n, nv=nv, dx=dx, u_hold=1)
    lat = Lattice(spec)
    u_dev = lat.flow_from_modes(tab)
    du = rel_l2(u_dev.cpu().numpy(), u_pre.cpu().numpy())
    f0 = torch.from_numpy(inputs.gaussian_ic(2, n, nv, dx, dv, ny=n)).cuda()
    a, b = f0.clone(), f0.clone()
    lat.step(a, u_pre, 4 * math.pi, 1e-4, dt, steps)
    lat.step(b, u_dev, 4 * math.pi, 1e-4, dt, steps)
    lat.sync()
    err = rel_l2(b.cpu().numpy(), a.cpu().numpy())
    say(f"  u rel L2 {du:.2e}; state after {steps} steps rel L2 {err:.2e}")
    assert du < 1e-6 and err < 1e-5
    lat.close()
