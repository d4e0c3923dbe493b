"""Short trajectories whose arrival times lie far apart on the grid, on both sides of the rule that lets windows of grid points gather
what such particles bring: few of them side by side, hundreds on top of each other, more windows than the rule's bins, some out
of the window, and one with an unusable sample.  Against the oracle, tolerances as in test_gpu_deposit.py."""
import numpy as np
import pytest
import torch

import oracle
from cases import synthetic

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
C = 299792458.0
TOL = {"fp64": 1e-9, "mixed": 2e-5}


def short(n_p, n_samples, n_pix, n_obs, points, spread, seed):
    """Particle k's points begin within `spread` of the grid (of 1: anywhere on it), `points` of them at pixel 0."""
    rng = np.random.default_rng(seed)
    c = synthetic(n_p=n_p, n_samples=n_samples, n_pix=n_pix, n_obs=16, seed=seed)
    c["r"] = c["r"] - c["r"][:, :1]
    tau, _, _ = oracle.eval_samples(0.0, c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"][:1], 0.0, 1.0)
    c["dt_obs"] = float(np.median(np.ptp(tau, axis=-1))) / points
    c["n_obs"] = n_obs
    begin = np.rint(spread * (n_obs - 1.1 * points) * rng.random(n_p)) + 0.37
    c["t0"] = float(np.min(tau))
    c["r"] = c["r"] - (begin * c["dt_obs"] * C)[:, None, None] * (c["x_det"][0] / np.linalg.norm(c["x_det"][0]))
    return c


def deposit(c, prec, geom, pixels=slice(None)):
    from paper_2206_03015_amd import lw
    t = {k: torch.as_tensor(np.ascontiguousarray(c[k]), device=DEV) for k in ("r", "beta", "beta_dot", "charge")}
    x_det = torch.as_tensor(np.ascontiguousarray(c["x_det"][pixels]), device=DEV)
    E, diag = lw.deposit_td(t["r"], t["beta"], t["beta_dot"], c["t_start"], c["dt"], x_det, c["t0"], c["dt_obs"], c["n_obs"],
                            prec=prec, geom=geom, charge=t["charge"])
    return E, diag.cpu().numpy()


@pytest.mark.parametrize("geom", ["exact", "farfield"])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n_p, n_samples, n_pix, n_obs, points, spread", [
    (4, 60, 70, 30001, 20000, 0.5),        # windows
    (300, 3, 2, 2000, 500, 0.0),           # one on top of the other
    (300, 3, 2, 2000, 500, 3.0),           # and two of three out of the window
    (12, 9, 2, 1025 * 512 + 7, 70000, 1.0),  # more windows than bins
    (700, 5, 33, 12000, 300, 1.0),
    (700, 5, 33, 60000, 3000, 1.0),        # particles of several lists
    (40, 2, 130, 9000, 2000, 0.5),         # two tiles
    (3, 1024, 3, 5000, 3000, 0.2),         # the longest
])
def test_both_sides_of_the_rule(n_p, n_samples, n_pix, n_obs, points, spread, prec, geom):
    c = short(n_p, n_samples, n_pix, n_obs, points, spread, seed=n_p + n_samples)
    c["beta"][1, n_samples // 2, 1] = np.nan
    E, diag = deposit(c, prec, geom)
    Eo, do = oracle.deposit_td(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], c["dt_obs"],
                               c["n_obs"], charge=c["charge"], geom=oracle.GEOM_EXACT if geom == "exact" else oracle.GEOM_FARFIELD)
    assert diag.tolist() == list(do) and do[3] > 0
    assert np.max(np.abs(E.double().cpu().numpy() - Eo)) <= TOL[prec] * np.max(np.abs(Eo))


def test_passes_of_pixels_decide_for_themselves():
    """More pixels than one pass takes: the last pass's twenty beside the first one's thousands."""
    n_pix, cut = 16384 + 20, 16384
    c = short(3, 4, n_pix, 4096, 3000, 0.3, seed=7)
    E, diag = deposit(c, "mixed", "exact")
    parts = [deposit(c, "mixed", "exact", s) for s in (slice(0, cut), slice(cut, None))]
    assert (diag == parts[0][1] + parts[1][1]).all() and diag[3] > 0
    for s, (Ep, _) in zip((slice(0, cut), slice(cut, None)), parts):
        assert float((E[s] - Ep).abs().max()) <= TOL["mixed"] * float(Ep.abs().max())
