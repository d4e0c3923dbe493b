"""Trajectories of a few samples on both sides of the rule that takes a step point by point or pixel by pixel (0.6 grid points per
interval of a whole step: 153 of a pixel in mixed precision, 76 in FP64), up to more points in an interval than its counters
hold (2^20), and in groups of several particles.  Against the oracle, tolerances as in test_gpu_deposit.py."""
import numpy as np
import pytest
import torch

import oracle
from cases import synthetic

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def check(c, prec):
    from paper_2206_03015_amd import lw
    t = {k: torch.as_tensor(np.ascontiguousarray(c[k]), device=DEV) for k in ("r", "beta", "beta_dot", "x_det", "charge")}
    E, diag = lw.deposit_td(t["r"], t["beta"], t["beta_dot"], c["t_start"], c["dt"], t["x_det"], c["t0"], c["dt_obs"],
                            c["n_obs"], prec=prec, charge=t["charge"])
    Eo, do = oracle.deposit_td(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], c["dt_obs"],
                               c["n_obs"], charge=c["charge"])
    assert diag.cpu().tolist() == list(do) and do[3] > 0
    assert np.max(np.abs(E.double().cpu().numpy() - Eo)) <= {"fp64": 1e-9, "mixed": 2e-5}[prec] * np.max(np.abs(Eo))


def short(n_p, n_samples, n_pix, points):
    """All start from one point, so that the window holds `points` grid points of particle 0's at pixel 0; its first and
    last arrival times lie between grid points (on one, the last bit of either side would decide)."""
    c = synthetic(n_p=n_p, n_samples=n_samples, n_pix=n_pix, n_obs=16, seed=n_samples)
    c["r"] = c["r"] - c["r"][:, :1]
    tau, _, _ = oracle.eval_samples(0.0, c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"][:1], 0.0, 1.0)
    c["dt_obs"] = float(np.ptp(tau[0, 0])) / points
    c["t0"] = float(np.min(tau)) - 2.37 * c["dt_obs"]
    c["n_obs"] = 2 * points + 4
    return c


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n_samples", [2, 3, 40])
@pytest.mark.parametrize("points", [1, 70, 80, 150, 160, 3000])
def test_around_the_dense_rule(points, n_samples, prec):
    check(short(3, n_samples, 70, points), prec)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_more_points_than_a_counter_holds(prec):
    check(short(1, 2, 2, (1 << 20) + 12345), prec)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n_p, n_samples", [(9000, 2), (4200, 30)])
def test_groups_of_short_trajectories(n_p, n_samples, prec):
    check(short(n_p, n_samples, 130, 20), prec)
