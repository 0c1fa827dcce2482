"""Host-side behaviour of bench.py that needs no GPU."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_bench_refuses_more_than_one_gpu():
    """The step runs on one MI355X; a multi-GPU request ends with a message
    (exit status 2) before anything touches a device."""
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "exactly one GPU" in r.stderr
    assert r.stdout == ""


def test_bench_refuses_a_multi_rank_launch():
    env = dict(os.environ, WORLD_SIZE="8")
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py")], capture_output=True,
                       text=True, timeout=120, env=env)
    assert r.returncode == 2 and "exactly one GPU" in r.stderr


def test_roofline_follows_the_launches_that_were_made():
    """Bytes per sweep from the mix of launches, not from the longest kind."""
    import bench
    p = dict(nx=1000, ny=100, nz=10, precision="fp32", poisson_scheme="chebyshev")
    # 25 sweeps between tests: 7 launches of three and 2 of two, and a test's own
    r = bench.sweep_roofline(p, 1e-3, (0, [1, 2, 7], 64))
    sweeps = 1 + 2 * 2 + 7 * 3
    assert r["bytes_per_sweep"] * sweeps == (16 + 9 * 20) * 1e6
    assert r["sweeps_per_launch"] == sweeps / 10 and r["kernel"] == "msweep_kernel<float, 3>"
    assert abs(r["achieved"] - r["bytes_per_sweep"] / 1e-3 / 1e9) < 1e-12
    r = bench.sweep_roofline(p, 1e-3, (0, [25, 0, 0], 0))
    assert r["bytes_per_sweep"] == 16e6 and r["kernel"] == "sweep1_kernel<float>"
    r = bench.sweep_roofline(p, 1e-3, (0, [1, 12, 0], 4))
    assert r["kernel"] == "sweep2_kernel<float>"
    r = bench.sweep_roofline(p, 1e-3, (3, [0, 0, 0], 64))
    assert r["bound"] == "fp64" and r["flops_per_sweep"] == 18e6
    before = dict(resident_passes=2, launches=[1, 2, 3], gave_up=0, refused=0, tile_rows=64)
    after = dict(before, resident_passes=5, launches=[1, 4, 9])
    assert bench.solver_runs(before, after) == (3, [0, 2, 6], 64)
