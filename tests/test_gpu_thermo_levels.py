"""Thermodynamics on planes that do not fill the blocks: cells taken in order
across levels, against the oracle, and at no higher cost than in square levels."""
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


def fields(shape, precision):
    rng = np.random.default_rng(3)
    thl, qt = rng.uniform(287.0, 291.0, shape), rng.uniform(5e-3, 14e-3, shape)
    if precision == "fp32":
        thl, qt = (f.astype(np.float32).astype(np.float64) for f in (thl, qt))
    return thl, qt


def params(shape, precision):
    nz, ny, nx = shape
    return li.workload("C1m", nx=nx, ny=ny, nz=nz, dz=800.0 / nz, precision=precision)


# (nz, ny, nx): by levels (few blocks, or planes that fill theirs), in order
# (more blocks, of 65 to 251 cells or a ragged last one)
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(2048, 4, 4), (2049, 4, 4), (2100, 1, 2), (512, 1, 65), (513, 1, 65),
                                   (171, 17, 31), (520, 1, 253), (520, 4, 63), (300, 17, 17),
                                   (4, 1, 70)])
def test_thermo_matches_oracle(gpu, oracle_lib, shape, precision):
    import torch
    p = params(shape, precision)
    thl, qt = fields(shape, precision)
    o = oracle_lib.thermo(p, thl, qt)
    g = gpu.LES(p).thermo(torch.from_numpy(thl), torch.from_numpy(qt))
    assert 0.2 < (o["ql"] > 0).mean() < 0.95
    tol = 1e-12 if precision == "fp64" else 1e-6
    for k in ("T", "ql", "b"):
        got = g[k].double().cpu().numpy()
        assert np.linalg.norm(got - o[k]) <= tol * np.linalg.norm(o[k]), k


def test_small_planes_cost_no_more_than_square_ones(gpu):
    """The same cells in planes of 4 x 4: within twice the time of 126 x 127
    planes (a block to each level took three times)."""
    import time
    import torch
    took = []
    for shape in ((60000, 4, 4), (60, 126, 127)):
        sim = gpu.LES(params(shape, "fp32"))
        thl, qt = (torch.from_numpy(f).to("cuda", torch.float32) for f in fields(shape, "fp32"))
        sim.thermo(thl, qt)
        best = 1e9
        for _ in range(20):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sim.thermo(thl, qt)
            torch.cuda.synchronize()
            best = min(best, time.perf_counter() - t0)
        sim.close()
        took.append(best)
    assert took[0] <= 2.0 * took[1], took
