"""The residual of a returned iterate on few x rows, one to a block, and on
more, four to a block: against FP64 on the host."""
import numpy as np
import pytest

import les_inputs as li

pytestmark = pytest.mark.gpu


# (nz, ny, nx): 4 to 520 rows, about the 128 where the blocks change too
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(4, 1, 70), (9, 1, 300), (16, 8, 33), (128, 1, 20), (129, 1, 20),
                                   (27, 19, 65), (10, 13, 9)])
def test_residual_of_a_kept_guess(precision, shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_04698_amd import les
    nz, ny, nx = shape
    p = li.workload("C1", nx=nx, ny=ny, nz=nz, dz=min(10.0, 8000.0 / nz), precision=precision,
                    mean_mode="swept", poisson_scheme="chebyshev")
    dt = np.float64 if precision == "fp64" else np.float32
    rhs = li.random_field(shape, seed=70).astype(dt)
    guess = (100.0 * li.random_field(shape, seed=71)).astype(dt)
    sim = les.LES(p)
    phi, st, rc = sim.poisson_solve(torch.from_numpy(rhs), phi=torch.from_numpy(guess).cuda(),
                                    use_guess=True, fixed_sweeps=3)
    f = phi.cpu().numpy().astype(np.float64)
    b = rhs.astype(np.float64)
    b = (b - b.mean()).astype(dt).astype(np.float64)
    e = np.concatenate([f[:1], f, f[-1:]])
    lap = ((np.roll(f, 1, 2) + np.roll(f, -1, 2) - 2 * f) / p["dx"] ** 2
           + (np.roll(f, 1, 1) + np.roll(f, -1, 1) - 2 * f) / p["dy"] ** 2
           + (e[2:] + e[:-2] - 2 * f) / p["dz"] ** 2)
    # the centred right-hand side is stored in the field's type; the iterate
    # returned is centred after the residual, which takes out no constant
    tol = 1e-11 if precision == "fp64" else 1e-5
    assert st["res_norm"] == pytest.approx(np.linalg.norm(b - lap), rel=tol)
