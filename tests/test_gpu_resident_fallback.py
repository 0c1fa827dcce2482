"""Resident passes that cannot be used: one whose launch is refused, one that
gives up a wait (a block is told from the host not to wait; every block still
runs to its end).  The solve is repeated launch by launch and ends as one that
ran so from the start, bit for bit; and tags that are used up start over."""
import numpy as np
import pytest

import les_inputs as li

pytestmark = pytest.mark.gpu

SHAPE = (20, 12, 70)  # 20 blocks


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_04698_amd import les
    les.load()
    return les


def make(gpu, precision, mean_mode, S, shape=SHAPE):
    nz, ny, nx = shape
    return gpu.LES(li.workload("C1", nx=nx, ny=ny, nz=nz, precision=precision,
                               mean_mode=mean_mode, poisson_scheme="chebyshev", poisson_tol=1e-4,
                               poisson_max_sweeps=600, poisson_check_every=7,
                               sweeps_per_launch=S))


def starts(sim, rhs):
    """(guess, use_guess, budget, fixed): none, kept, kept and gated, dropped,
    over its budget, ending in the storage precision's reach, a fixed count."""
    import torch
    exact, _, _ = sim.poisson_solve(rhs)
    noise = torch.from_numpy(li.random_field(SHAPE, seed=6)).to(exact)
    near = (exact + 1e-2 * exact.abs().max().item() * noise).contiguous()
    return [(None, False, 0, 0), (near, True, 0, 0), (near, 2, 400, 0), (1e3 * near, 2, 400, 0),
            (near, 2, 7, 0), (exact, 2, 50, 0), (near, True, 0, 9), (None, False, 0, 31)]


def solve(sim, rhs, start):
    guess, mode, budget, fixed = start
    phi, st, rc = sim.poisson_solve(rhs, phi=None if guess is None else guess.clone(),
                                    use_guess=mode, budget=budget, fixed_sweeps=fixed)
    return phi.cpu().numpy(), rc, [st[k] for k in ("sweeps", "status", "guess", "guess_sweeps")], st


@pytest.mark.parametrize("fault", ["refused", "wait"])
@pytest.mark.parametrize("precision,mean_mode", [("fp32", "exact"), ("fp64", "exact"),
                                                 ("fp32", "swept"), ("fp64", "level")])
def test_solve_is_repeated_launch_by_launch(gpu, precision, mean_mode, fault):
    import torch
    rhs = torch.from_numpy(li.random_field(SHAPE, seed=5))
    plain = make(gpu, precision, mean_mode, 1)
    which = {"refused": gpu.LES_FAULT_REFUSED, "wait": gpu.LES_FAULT_WAIT}[fault]
    flags = set()
    for i, start in enumerate(starts(plain, rhs)):
        want = solve(plain, rhs, start)
        flags.add(want[2][2])
        again = want[2][2] in (3, 4)  # the solve has a second pass
        for after in (0, 1) if again else (0,):
            print(f"{fault} {precision} {mean_mode} start {i} after {after}", flush=True)
            sim = make(gpu, precision, mean_mode, 0)
            sim.resident_fault(which, after)
            got = solve(sim, rhs, start)
            state = sim.solver_state()
            assert state["resident_blocks"] == 0 and state["resident_passes"] == after
            assert (state["refused"], state["gave_up"]) == ((1, 0) if fault == "refused" else (0, 1))
            assert sum(state["launches"]) > 0
            more = solve(sim, rhs, start)  # the handle goes on launch by launch
            assert sim.solver_state()["resident_passes"] == after
            sim.close()
            for g in (got, more):
                assert np.array_equal(g[0], want[0])
                assert g[1:3] == want[1:3]
                # sums of the residual over another decomposition
                assert g[3]["res_norm"] == pytest.approx(want[3]["res_norm"], rel=1e-12)
                assert g[3]["rhs_norm"] == want[3]["rhs_norm"]
    assert flags >= {0, 1, 2, 3}


@pytest.mark.parametrize("fault", ["refused", "wait"])
def test_nonfinite_rhs_after_a_fault(gpu, fault):
    import torch
    sim = make(gpu, "fp64", "exact", 0)
    rhs = torch.from_numpy(li.random_field(SHAPE, seed=5)).to("cuda")
    bad = rhs.clone()
    bad[3, 4, 5] = float("inf")
    sim.resident_fault({"refused": 1, "wait": 2}[fault])
    with pytest.raises(gpu.LesError) as e:
        sim.poisson_solve(bad)
    assert e.value.code == gpu.LES_ERR_NONFINITE
    phi, st, rc = sim.poisson_solve(rhs)
    assert rc == 0 and st["res_norm"] <= 1e-4 * st["rhs_norm"]


@pytest.mark.parametrize("shape", [SHAPE, (64, 64, 64), (40, 1, 100)])
def test_used_up_tags_start_over(gpu, shape):
    """The words still hold the first solves' tags when the numbers start
    over: uncleared they would be taken for the new solve's."""
    import torch
    rhs = torch.from_numpy(li.random_field(shape, seed=8))
    plain, sim = make(gpu, "fp32", "exact", 1, shape), make(gpu, "fp32", "exact", 0, shape)
    most = 2 ** 32 - 1
    for fixed, tag in ((38, 0), (25, 0), (38, most - (38 + 4)),  # the last numbers that fit
                       (38, 0), (25, most - (25 + 3)),           # one too few: starts over
                       (38, 0), (38, most), (25, 0)):
        sim.resident_fault(next_tag=tag)
        a, b = plain.poisson_solve(rhs, fixed_sweeps=fixed), sim.poisson_solve(rhs, fixed_sweeps=fixed)
        assert np.array_equal(a[0].cpu().numpy(), b[0].cpu().numpy())
    got = sim.solver_state()
    assert (got["resident_passes"], got["gave_up"]) == (8, 0)


def test_fault_arguments_are_checked(gpu):
    sim = make(gpu, "fp32", "exact", 0)
    for bad in (dict(fault=3), dict(fault=-1), dict(fault=1, after=-1)):
        with pytest.raises(gpu.LesError) as e:
            sim.resident_fault(**bad)
        assert e.value.code == gpu.LES_ERR_ARG
    sim.resident_fault(next_tag=1000)
    with pytest.raises(gpu.LesError) as e:
        sim.resident_fault(next_tag=999)
    assert e.value.code == gpu.LES_ERR_ARG
