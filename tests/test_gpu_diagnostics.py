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


def centred(f, ax, d):
    return (np.roll(f, -1, ax) - np.roll(f, 1, ax)) / (2.0 * d)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(4, 1, 51200), (16, 1, 4097), (4, 2, 3000), (9, 3, 1027),
                                   (64, 200, 4), (5, 33, 2), (6, 17, 16), (4, 40, 17), (4, 9, 32),
                                   (4, 70, 33)])
def test_pieces_of_rows_and_rows_side_by_side(precision, shape):
    """Levels of few rows (rows in pieces) and of narrow rows (several to a
    wave): every sum, the divergence and the maxima against FP64 on the host."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_04698_amd import les
    nz, ny, nx = shape
    dt = np.float64 if precision == "fp64" else np.float32
    p = li.workload("C1", nx=nx, ny=ny, nz=nz, dz=5.0, precision=precision)
    st = {k: li.random_field(shape, seed=60 + q) for q, k in enumerate("uvw")}
    st["thl"] = 300.0 + 0.1 * li.random_field(shape, seed=64)
    st["qt"] = 1e-3 * (1.0 + 0.1 * li.random_field(shape, seed=65))
    st["p"] = np.zeros(shape)
    st = {k: np.ascontiguousarray(v.astype(dt)) for k, v in st.items()}
    sim = les.LES(p, {k: torch.from_numpy(v) for k, v in st.items()})
    d = sim.diagnostics()
    sim.close()
    f = {k: v.astype(np.float64) for k, v in st.items()}
    for name in ("thl", "qt", "u", "v", "w"):
        tol = 1e-13 * np.abs(f[name]).mean((1, 2)).max()
        assert np.abs(d["profiles"][name] - f[name].mean((1, 2))).max() <= tol, name
    # the reference state of Sec. 2.1 at the level centres
    z = (np.arange(nz) + 0.5) * p["dz"]
    p0 = p["p00"] * (1.0 - p["g"] * z / (p["cpd"] * p["theta0"])) ** (p["cpd"] / p["Rd"])
    T0 = p["theta0"] * (p0 / p["p00"]) ** (p["Rd"] / p["cpd"])
    rho = (p0 / (p["Rd"] * T0))[:, None, None]
    rw = rho * f["w"]
    div = (centred(rho * f["u"], 2, p["dx"]) + (centred(rho * f["v"], 1, p["dy"]) if ny > 1 else 0)
           + (np.concatenate([rw[1:], -rw[-1:]]) - np.concatenate([-rw[:1], rw[:-1]]))
           / (2.0 * p["dz"]))
    vol = p["dx"] * p["dy"] * p["dz"]
    cfl = (np.abs(f["u"]) * p["dt"] / p["dx"] + np.abs(f["v"]) * p["dt"] / p["dy"]
           + np.abs(f["w"]) * p["dt"] / p["dz"]).max()
    # FP64 throughout, at most 3e5 terms in two orders
    for key, want in (("div_max", np.abs(div).max()), ("cfl", cfl),
                      ("div_l2", np.sqrt((div ** 2).sum())),
                      ("ke", 0.5 * (rho * (f["u"] ** 2 + f["v"] ** 2 + f["w"] ** 2)).sum() * vol),
                      ("mass_thl", (rho * f["thl"]).sum() * vol),
                      ("mass_qt", (rho * f["qt"]).sum() * vol)):
        assert d[key] == pytest.approx(want, rel=1e-12), key


def test_one_row_costs_no_more_than_square_levels():
    """The same number of cells in one row of a level: within four times the
    square level's time (it took 30 times with a row to one wave)."""
    import time
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_04698_amd import les
    took = []
    for nz, ny, nx in ((16, 1, 51200), (16, 226, 226)):
        sim = les.LES(li.workload("C1", nx=nx, ny=ny, nz=nz, dz=5.0, precision="fp64"))
        sim.diagnostics()
        best = 1e9
        for _ in range(20):
            t0 = time.perf_counter()
            sim.diagnostics()
            best = min(best, time.perf_counter() - t0)
        sim.close()
        took.append(best)
    assert took[0] <= 4.0 * took[1], took
