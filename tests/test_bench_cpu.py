"""bench.py's host-side contract (no GPU): one GPU only, argument checks,
the step-kernel naming and the counter-validity hash."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _bench(*args):
    return subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"),
                           *args], capture_output=True, text=True, timeout=120,
                          cwd=ROOT)


def test_more_than_one_gpu_exits_with_a_message():
    r = _bench("--gpus", "2")
    assert r.returncode == 2
    assert "single" in r.stderr and "--gpus 1" in r.stderr
    assert r.stdout == ""


def test_non_positive_stokes_number_is_refused():
    r = _bench("--st", "0", "--workload", "coarse-mlp-256x256")
    assert r.returncode != 0 and "--st" in r.stderr


def test_step_kernel_names_follow_the_library_dispatch():
    sys.path.insert(0, ROOT)
    import bench
    assert bench.step_kernel(2, 512, 33, "f32") == "k_step2d"
    assert bench.step_kernel(1, 16384, 129, "f32") == "k_step1d_parts"
    assert bench.step_kernel(1, 256, 33, "f64") == "k_step1d_parts"
    assert bench.step_kernel(1, 1 << 20, 33, "f32") == "k_step1d"
    assert bench.step_kernel(1, 4096, 129, "f64") == "k_step1d"
    assert bench.step_kernel(1, 4096, 9, "f32") == "k_step1d"


def test_named_kernels_and_launches_follow_the_library_rules():
    """Calls of several steps and of several sub-steps: the kernel named and
    the launches counted are those of the library's own rules, asked of it
    directly (they are host code)."""
    sys.path.insert(0, ROOT)
    import ctypes

    import bench
    from paper_1508_02899_amd.lattice import load_library
    lib = load_library()
    multi = getattr(lib, "_ZN3lat18step1d_multi_stepsEiliii")
    multi.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_int] * 3

    class Dims(ctypes.Structure):
        _fields_ = [(k, ctypes.c_int) for k in ("nv", "f64", "koren")] + [
            (k, ctypes.c_int64) for k in ("nx", "ny", "pitch")]

    take = getattr(lib, "_ZN3lat15step2d_sub_takeERKNS_12lattice_dimsEl")
    take.argtypes = [ctypes.POINTER(Dims), ctypes.c_int64]
    for nv in (3, 5, 7, 9, 11, 13, 17, 21, 25, 33, 65, 129):
        for n in (1, 256, 8192, 8193, 16384, 32768, 32769, 65536, 65537):
            for dtype in ("f32", "f64"):
                for nsub in (1, 2, 3, 5, 10, 11):
                    for shift in (1, 2, 16):
                        assert bench.steps_per_launch(
                            n, nv, dtype, nsub, shift) == multi(
                            nv, n, shift, nsub, dtype == "f64"), (nv, n)
    for w in bench.WORKLOADS.values():
        if w["dim"] != 2:
            continue
        n, nv = w["n"], w["nv"]
        for scheme in ("koren", "upwind"):
            for nsub in range(1, 9):
                d = Dims(nv, 0, scheme == "koren", n, n, n * n)
                got = bench.sub_steps_per_pass(n, nv, "f32", nsub, scheme)
                assert got == take(ctypes.byref(d), nsub), (n, nv, nsub)
    assert bench.step_kernel(1, 256, 33, "f64", 1000) == "k_step1d_multi"
    assert bench.step_launches(1, 256, 33, "f64", 1000) == 250
    assert bench.step_kernel(1, 16384, 129, "f32", 1000) == "k_step1d_parts"
    assert bench.step_launches(1, 16384, 129, "f32", 1000) == 1000
    assert bench.step_kernel(2, 512, 33, "f32", 200, 2) == "k_step2d_sub"
    assert bench.step_launches(2, 512, 33, "f32", 200, 3) == 400


def test_recorded_counters_match_the_kernel_sources():
    """Every traffic file under profiles/ names the workload, its kernel and
    the hash of the sources it was taken on; a file whose hash matches is
    the one bench.py reports, and its bytes are close to the algorithmic
    bytes (no re-reads reach HBM)."""
    sys.path.insert(0, ROOT)
    import bench
    d = os.path.join(ROOT, "profiles")
    files = [f for f in os.listdir(d) if f.startswith("traffic_")]
    assert files
    for f in files:
        with open(os.path.join(d, f)) as fh:
            t = json.load(fh)
        w = bench.WORKLOADS[t["workload"]]
        if w.get("batch"):
            assert t["kernel_hash"] == bench.kernel_hash("batch"), f
            assert (bench.load_traffic(t["workload"], "batch") ==
                    t["bytes_per_step"])
        else:
            assert t["kernel_hash"] == bench.kernel_hash(w["dim"]), f
            assert bench.load_traffic(t["workload"]) == t["bytes_per_launch"]
        # the lattice passes re-read nothing; the batched kernel re-reads
        # tile edges that two workgroups share (its paired chunks trade
        # about 8 % more reads for shorter steps)
        top = 1.10 if w.get("batch") else 1.05
        assert 0.99 < t["traffic_over_algorithmic"] < top, f
