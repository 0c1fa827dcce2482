"""Horizontal sums of the diagnostics on grids whose levels are split over
several blocks, against FP64 sums on the host: fewer rows than waves, rows that
do not fill a wave, one and several parts, one row."""
import numpy as np
import pytest

import les_inputs as li

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(4, 1, 2), (4, 2, 3), (5, 3, 65), (33, 19, 64), (7, 130, 100),
                                   (4, 700, 70), (640, 1, 129)])
def test_profiles_and_integrals_match_host_sums(precision, shape):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_04698_amd import les
    nz, ny, nx = shape
    dt = np.float64 if precision == "fp64" else np.float32
    p = li.workload("C1", nx=nx, ny=ny, nz=nz, dz=min(5.0, 2000.0 / nz), precision=precision)
    st = {k: li.random_field(shape, seed=40 + q) for q, k in enumerate("uvw")}
    st["thl"] = 300.0 + 0.1 * li.random_field(shape, seed=44)
    st["qt"] = 1e-3 * (1.0 + 0.1 * li.random_field(shape, seed=45))
    st["p"] = np.zeros(shape)
    st = {k: np.ascontiguousarray(v.astype(dt)) for k, v in st.items()}
    sim = les.LES(p, {k: torch.from_numpy(v) for k, v in st.items()})
    d = sim.diagnostics()
    sim.close()
    f = {k: v.astype(np.float64) for k, v in st.items()}
    want = dict(thl=f["thl"], qt=f["qt"], u=f["u"], v=f["v"], w=f["w"], ww=f["w"] ** 2,
                www=f["w"] ** 3)
    got = d["profiles"]
    # FP64 sums of at most 1e5 terms in two orders, relative to their magnitudes
    for name, w in want.items():
        key = {"ww": "w2", "www": "w3"}.get(name, name)
        assert np.abs(got[key] - w.mean((1, 2))).max() <= 1e-13 * np.abs(w).mean((1, 2)).max(), name
    cfl = (np.abs(f["u"]) * p["dt"] / p["dx"] + np.abs(f["v"]) * p["dt"] / p["dy"]
           + np.abs(f["w"]) * p["dt"] / p["dz"]).max()
    assert d["cfl"] == pytest.approx(cfl, rel=1e-14)
