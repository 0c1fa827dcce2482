"""Launches of two and three sweeps against one by one, on grids that are too
large to be resident on the chip: the same iterates bit for bit and the same
stopping sweep, with ragged tiles and one and several z chunks."""
import numpy as np
import pytest

import les_inputs as li

pytestmark = pytest.mark.gpu

# (nz, ny, nx): more than 256 boxes of 64 x 16 x 8 (Jacobi), of 64 x 16 x 32
# (Chebyshev; FP64 half the levels)
CASES = [("fp32", "jacobi", (64, 100, 300)), ("fp64", "jacobi", (64, 100, 300)),
         ("fp32", "chebyshev", (70, 33, 2100)), ("fp64", "chebyshev", (70, 33, 2100)),
         ("fp64", "chebyshev", (5, 500, 3000)), ("fp32", "chebyshev", (4, 2500, 1700)),
         ("fp32", "chebyshev", (135, 180, 530)), ("fp32", "chebyshev", (9, 70, 15000))]


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_04698_amd import les
    les.load()
    return les


@pytest.mark.parametrize("precision,scheme,shape", CASES)
def test_sweeps_of_a_launch_bitwise_equal(gpu, precision, scheme, shape):
    import torch
    nz, ny, nx = shape
    print(f"several sweeps per launch {precision} {scheme} {nx}x{ny}x{nz}", flush=True)
    rhs = torch.from_numpy(li.random_field(shape, seed=19))
    got = []
    for S in (1, 2, 0):
        p = li.workload("C1", nx=nx, ny=ny, nz=nz, precision=precision, poisson_scheme=scheme,
                        poisson_tol=1e-3, poisson_max_sweeps=120, poisson_check_every=11,
                        sweeps_per_launch=S)
        sim = gpu.LES(p)
        out = []
        for fixed in (1, 2, 3, 5, 22, 0):  # 0: to the tolerance, or the cap
            phi, st, rc = sim.poisson_solve(rhs, fixed_sweeps=fixed)
            out.append((phi.cpu().numpy(), st["sweeps"], st["status"], st["res_norm"]))
        got.append(out)
        sim.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a[0], b[0])
            assert a[1:3] == b[1:3]
            # the residual's FP64 sum is taken over another decomposition
            assert b[3] == pytest.approx(a[3], rel=1e-12)
