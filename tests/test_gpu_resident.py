"""Solves resident on the chip against the one-sweep launches: the same
iterates bit for bit and the same stopping sweep, at the edges of every box
shape (one box, a box per direction, ragged columns, rows and levels, boxes
that neighbour themselves through the periodic wrap)."""
import numpy as np
import pytest

import les_inputs as li

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_04698_amd import les
    les.load()
    return les


# (nz, ny, nx): small boxes hold 64 x 8 x 4 cells (one row: 64 x 1 x 32),
# medium ones 64 x 16 x 4 and x 8, large ones 64 x 16 x 16 and, in FP32, x 32
# (one row: 64 x 1 x 256), at most 256 boxes of a shape
SMALL = [(4, 8, 64), (8, 16, 128), (4, 2, 2), (5, 3, 3), (33, 20, 130), (32, 32, 32), (7, 9, 65),
         (61, 75, 100)]
MEDIUM = [(64, 128, 256), (50, 90, 150), (50, 120, 250), (16, 256, 256)]
LARGE = {"fp32": [(128, 256, 256), (100, 200, 250), (120, 33, 1000), (64, 256, 256),
                  (100, 120, 250)],
         "fp64": [(64, 256, 256), (70, 130, 200)]}
ROWS = [(32, 1, 64), (8, 1, 2), (9, 1, 65), (128, 1, 1024), (256, 1, 256), (250, 1, 2100),
        (640, 1, 5120)]
CASES = ([(p, s, shape) for p in ("fp32", "fp64") for s in ("jacobi", "chebyshev")
          for shape in SMALL + MEDIUM + ROWS[:4]]
         + [(p, "chebyshev", shape) for p in ("fp32", "fp64") for shape in LARGE[p] + ROWS[4:]])


@pytest.mark.parametrize("precision,scheme,shape", CASES)
def test_resident_solve_bitwise_equal(gpu, precision, scheme, shape):
    import torch
    nz, ny, nx = shape
    print(f"resident solve {precision} {scheme} {nx}x{ny}x{nz}", flush=True)
    rhs = torch.from_numpy(li.random_field(shape, seed=17))
    got = []
    for S in (1, 0):
        p = li.workload("C1", nx=nx, ny=ny, nz=nz, precision=precision, poisson_scheme=scheme,
                        poisson_tol=1e-4, poisson_max_sweeps=600, poisson_check_every=7,
                        sweeps_per_launch=S)
        sim = gpu.LES(p)
        out = []
        for fixed in (1, 38, 0):  # 0: to the tolerance, or the cap
            phi, st, rc = sim.poisson_solve(rhs, fixed_sweeps=fixed)
            out.append((phi.cpu().numpy(), st["sweeps"], st["status"], st["res_norm"]))
        got.append(out)
        sim.close()
    for a, b in zip(*got):
        assert np.array_equal(a[0], b[0])
        assert a[1:3] == b[1:3]
        # the residual's FP64 sum is taken over another decomposition
        assert b[3] == pytest.approx(a[3], rel=1e-12)


def test_resident_solve_of_zero_and_nonfinite_rhs(gpu):
    import torch
    p = li.workload("C1", nx=64, ny=16, nz=8, poisson_scheme="chebyshev")
    sim = gpu.LES(p)
    rhs = torch.zeros((8, 16, 64), dtype=torch.float64, device="cuda")
    phi, st, rc = sim.poisson_solve(rhs)
    assert st["sweeps"] == 0 and not phi.any()
    rhs[1, 2, 3] = float("nan")
    with pytest.raises(gpu.LesError) as e:
        sim.poisson_solve(rhs)
    assert e.value.code == gpu.LES_ERR_NONFINITE
    # and the handle solves again
    phi, st, rc = sim.poisson_solve(torch.from_numpy(li.random_field((8, 16, 64), seed=1)))
    assert rc == 0 and st["res_norm"] <= p["poisson_tol"] * st["rhs_norm"]


@pytest.mark.parametrize("precision,mean_mode", [("fp32", "exact"), ("fp64", "exact"),
                                                 ("fp32", "swept"), ("fp64", "level")])
def test_resident_solve_with_a_guess_bitwise_equal(gpu, precision, mean_mode):
    """The gate, the sweep budget and the repeat after it are taken on the
    device before the sweeps' outcome is known to the host: the same iterate
    and the same counts as launch by launch, for a guess that is kept, one
    that is dropped and one whose budget is too short."""
    import torch
    shape = (20, 12, 70)
    rhs = torch.from_numpy(li.random_field(shape, seed=5))
    noise = torch.from_numpy(li.random_field(shape, seed=6))
    got = []
    for S in (1, 0):
        p = li.workload("C1", nx=70, ny=12, nz=20, precision=precision, mean_mode=mean_mode,
                        poisson_scheme="chebyshev", poisson_tol=1e-4, poisson_max_sweeps=600,
                        poisson_check_every=7, sweeps_per_launch=S)
        sim = gpu.LES(p)
        exact, st, rc = sim.poisson_solve(rhs)
        assert rc == 0
        scale = exact.abs().max().item()
        near = (exact + 1e-2 * scale * noise.to(exact)).contiguous()
        out = []
        for guess, mode, budget, fixed in ((near, True, 0, 0), (near, 2, 400, 0),
                                           (1e3 * near, 2, 400, 0), (near, 2, 7, 0),
                                           (exact, 2, 50, 0), (near, True, 0, 5)):
            phi, st, rc = sim.poisson_solve(rhs, phi=guess.clone(), use_guess=mode,
                                            budget=budget, fixed_sweeps=fixed)
            out.append((phi.cpu().numpy(), [st[k] for k in ("sweeps", "status", "guess",
                                                            "guess_sweeps")], st["res_norm"]))
        got.append(out)
        sim.close()
    print([o[1] for o in got[0]])
    assert {o[1][2] for o in got[0]} >= {1, 2, 3}
    for a, b in zip(*got):
        assert np.array_equal(a[0], b[0])
        assert a[1] == b[1]
        assert b[2] == pytest.approx(a[2], rel=1e-12)


def test_resident_solves_of_two_threads(gpu):
    """Two handles on streams of their own, each driven by a thread: the
    solves' blocks fill the chip, and each solve ends as it does alone."""
    import threading
    import torch
    shapes = [(64, 64, 64), (64, 256, 256)]
    want, got = [None, None], [[], []]
    sims, rhs = [], []
    for q, shape in enumerate(shapes):
        nz, ny, nx = shape
        with torch.cuda.stream(torch.cuda.Stream()):
            p = li.workload("C1", nx=nx, ny=ny, nz=nz, precision="fp32",
                            poisson_scheme="chebyshev", poisson_tol=1e-4)
            sims.append(gpu.LES(p))
        rhs.append(torch.from_numpy(li.random_field(shape, seed=50 + q)))
        torch.cuda.synchronize()
        phi, st, rc = sims[q].poisson_solve(rhs[q], fixed_sweeps=100)
        want[q] = phi.cpu().numpy()

    def run(q):
        with torch.cuda.stream(sims[q].stream):
            for _ in range(8):
                phi, st, rc = sims[q].poisson_solve(rhs[q], fixed_sweeps=100)
                got[q].append(phi.cpu().numpy())

    threads = [threading.Thread(target=run, args=(q,)) for q in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for q in range(2):
        assert len(got[q]) == 8
        assert all(np.array_equal(a, want[q]) for a in got[q])
