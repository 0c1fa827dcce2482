"""Which way a solve ran, as the library reports it: the comparisons of the
resident and of the several-sweep kernels with the one-sweep launches hold
only where those kernels ran."""
import threading

import numpy as np
import pytest

import les_inputs as li
from test_gpu_multisweep import CASES as SEVERAL
from test_gpu_resident import CASES as RESIDENT

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_04698_amd import les
    les.load()
    return les


def workload(precision, scheme, shape, **kw):
    nz, ny, nx = shape
    return li.workload("C1", nx=nx, ny=ny, nz=nz, precision=precision, poisson_scheme=scheme,
                       poisson_tol=1e-4, poisson_max_sweeps=600, poisson_check_every=7, **kw)


# one row too small for the largest boxes: launch by launch
TOO_SMALL = (250, 1, 2100)


@pytest.mark.parametrize("precision,scheme,shape", [c for c in RESIDENT if c[2] != TOO_SMALL])
def test_resident_cases_run_resident(gpu, precision, scheme, shape):
    import torch
    print(f"resident {precision} {scheme} {shape}", flush=True)
    sim = gpu.LES(workload(precision, scheme, shape))
    plan = gpu.solver_plan(sim.cfg)
    assert plan["resident_blocks"] > 0
    rhs = torch.from_numpy(li.random_field(shape, seed=17))
    for fixed in (6, 38, 0):
        sim.poisson_solve(rhs, fixed_sweeps=fixed)
    got = sim.solver_state()
    assert got == dict(plan, resident_passes=3)


# the FP32 Jacobi entry of the shared list runs one sweep per launch; a grid
# well inside the rule for three takes its place here
ONE_BY_ONE = ("fp32", "jacobi", (64, 100, 300))


@pytest.mark.parametrize("precision,scheme,shape",
                         [c for c in SEVERAL if c != ONE_BY_ONE]
                         + [("fp32", "jacobi", (135, 180, 530))])
def test_several_sweeps_run_in_a_launch(gpu, precision, scheme, shape):
    import torch
    print(f"several sweeps per launch {precision} {scheme} {shape}", flush=True)
    rhs = torch.from_numpy(li.random_field(shape, seed=19))
    want = None
    for S, depth in ((1, 1), (2, 2), (0, 3)):
        sim = gpu.LES(workload(precision, scheme, shape, sweeps_per_launch=S))
        out = [sim.poisson_solve(rhs, fixed_sweeps=f)[0].cpu().numpy() for f in (1, 2, 3, 5, 22)]
        got = sim.solver_state()
        sim.close()
        assert got["resident_blocks"] == 0 and got["sweeps_per_launch"] == depth
        assert [n > 0 for n in got["launches"]][depth - 1:] == [True] + [False] * (3 - depth)
        want = want or out
        assert all(np.array_equal(a, b) for a, b in zip(want, out))


def test_resident_solves_of_two_threads_give_up_no_wait(gpu):
    import torch
    shapes = [(64, 64, 64), (64, 256, 256)]
    sims, rhs = [], []
    for q, shape in enumerate(shapes):
        with torch.cuda.stream(torch.cuda.Stream()):
            sims.append(gpu.LES(workload("fp32", "chebyshev", shape)))
        rhs.append(torch.from_numpy(li.random_field(shape, seed=50 + q)))

    def run(q):
        with torch.cuda.stream(sims[q].stream):
            for _ in range(8):
                sims[q].poisson_solve(rhs[q], fixed_sweeps=100)

    threads = [threading.Thread(target=run, args=(q,)) for q in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for sim in sims:
        got = sim.solver_state()
        assert (got["resident_passes"], got["gave_up"], got["refused"]) == (8, 0, 0)
        assert got["launches"] == [0, 0, 0]


@pytest.mark.parametrize("precision,scheme,shape", [
    ("fp32", "chebyshev", (500, 1, 4900)), ("fp64", "chebyshev", (500, 1, 4900)),
    ("fp64", "jacobi", (500, 1, 4900)), ("fp32", "chebyshev", (33, 338, 277))])
def test_ragged_large_boxes_bitwise_equal(gpu, precision, scheme, shape):
    """Large boxes that fill neither their columns nor their levels, on grids
    that are still faster resident."""
    import torch
    print(f"ragged large boxes {precision} {scheme} {shape}", flush=True)
    rhs = torch.from_numpy(li.random_field(shape, seed=23))
    out = []
    for S in (1, 0):
        sim = gpu.LES(workload(precision, scheme, shape, sweeps_per_launch=S))
        out.append([sim.poisson_solve(rhs, fixed_sweeps=f) for f in (6, 38, 0)])
        assert (sim.solver_state()["resident_passes"] == 3) == (S == 0)
        sim.close()
    for a, b in zip(*out):
        assert np.array_equal(a[0].cpu().numpy(), b[0].cpu().numpy())
        assert [a[1][k] for k in ("sweeps", "status")] == [b[1][k] for k in ("sweeps", "status")]


@pytest.mark.parametrize("precision,scheme,shape", [
    (p, s, shape) for p in ("fp32", "fp64") for s, shape in (
        ("chebyshev", (128, 1, 1024)), ("jacobi", (93, 1, 2100)), ("chebyshev", (64, 4, 2000)),
        ("chebyshev", (33, 6, 4000)), ("jacobi", (91, 5, 3171)))])
def test_thin_two_sweep_launches_bitwise_equal(gpu, precision, scheme, shape):
    """Two sweeps per launch in four-row waves: segments of 62 columns, rows
    and z chunks that do not divide the grid, tests at odd sweeps."""
    import torch
    print(f"thin two-sweep launches {precision} {scheme} {shape}", flush=True)
    rhs = torch.from_numpy(li.random_field(shape, seed=31))
    out = []
    for S in (1, 2):
        sim = gpu.LES(workload(precision, scheme, shape, sweeps_per_launch=S))
        out.append([sim.poisson_solve(rhs, fixed_sweeps=f) for f in (1, 2, 3, 22, 0)])
        got = sim.solver_state()
        assert got["tile_rows"] == (4 if S == 2 else 0) and (got["launches"][1] > 0) == (S == 2)
        sim.close()
    for a, b in zip(*out):
        assert np.array_equal(a[0].cpu().numpy(), b[0].cpu().numpy())
        assert [a[1][k] for k in ("sweeps", "status")] == [b[1][k] for k in ("sweeps", "status")]
        assert b[1]["res_norm"] == pytest.approx(a[1]["res_norm"], rel=1e-12)


@pytest.mark.parametrize("scheme,mean_mode", [("chebyshev", "exact"), ("jacobi", "swept")])
@pytest.mark.parametrize("rhs", ["zero", "constant", "nan", "inf"])
def test_fixed_count_without_a_right_hand_side_is_refused_either_way(gpu, rhs, scheme, mean_mode):
    """A fixed number of sweeps on a right-hand side that is nothing, or not
    finite: the same refusal resident and launch by launch; to the tolerance
    the first is solved by nothing."""
    import torch
    shape = (6, 10, 70)
    f = np.full(shape, {"zero": 0.0, "constant": 3.0}.get(rhs, 1.0))
    if rhs in ("nan", "inf"):
        f[2, 3, 4] = float(rhs)
    for S in (1, 2, 0):
        sim = gpu.LES(workload("fp32", scheme, shape, mean_mode=mean_mode, sweeps_per_launch=S))
        with pytest.raises(gpu.LesError) as e:
            sim.poisson_solve(torch.from_numpy(f), fixed_sweeps=5)
        assert e.value.code == gpu.LES_ERR_STATE
        if rhs in ("nan", "inf"):
            with pytest.raises(gpu.LesError) as e:
                sim.poisson_solve(torch.from_numpy(f))
            assert e.value.code == gpu.LES_ERR_NONFINITE
        else:
            phi, st, rc = sim.poisson_solve(torch.from_numpy(f))
            assert rc == 0 and st["sweeps"] == 0 and not phi.any()
        sim.close()


@pytest.mark.parametrize("mean_mode,least", [("exact", 1), ("level", 6), ("swept", 6)])
def test_small_fixed_counts_run_launch_by_launch(gpu, mean_mode, least):
    """A resident launch takes longer than the few sweeps it would save; with a
    guess or exact parts it saves a read-back too.  The iterates are the same
    either way."""
    import torch
    shape = (20, 12, 70)
    rhs = torch.from_numpy(li.random_field(shape, seed=37))
    one, sim = (gpu.LES(workload("fp64", "chebyshev", shape, mean_mode=mean_mode,
                                 sweeps_per_launch=S)) for S in (1, 0))
    for fixed in range(1, 9):
        seen = sim.solver_state()["resident_passes"]
        a, b = (s.poisson_solve(rhs, fixed_sweeps=fixed) for s in (one, sim))
        assert np.array_equal(a[0].cpu().numpy(), b[0].cpu().numpy())
        assert sim.solver_state()["resident_passes"] - seen == (fixed >= least)
        a, b = (s.poisson_solve(rhs, phi=0.5 * a[0], use_guess=True, fixed_sweeps=fixed)
                for s in (one, sim))
        assert np.array_equal(a[0].cpu().numpy(), b[0].cpu().numpy())
        assert sim.solver_state()["resident_passes"] - seen == (fixed >= least) + 1
