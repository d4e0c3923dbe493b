"""The careful path of lw_deposit_td at the ends of the 64 samples whose arrival-time coefficients are formed at a time: a
particle with an undefined sample beside one without, against the oracle (tolerances as in test_gpu_deposit.py)."""
import numpy as np
import pytest
import torch

import oracle
from cases import synthetic

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("geom, far", [("exact", False), ("exact", True), ("farfield", False)])
@pytest.mark.parametrize("n_samples, bad", [(2, 0), (63, 62), (64, 1), (65, 64), (128, 63), (129, 64), (200, 127)])
def test_careful_path(n_samples, bad, geom, far, prec):
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=3, n_samples=n_samples, n_pix=70, n_obs=150, seed=n_samples, dt=2e-18 * 700 / max(n_samples, 200))
    if far:  # pixels at several distances: each takes its own arrival-time form
        c["x_det"] = c["x_det"] * np.linspace(0.5, 3.0, 70)[:, None]
    c["beta_dot"] = c["beta_dot"].copy()
    c["beta_dot"][1, bad, 2] = np.inf
    t = {k: torch.as_tensor(np.ascontiguousarray(c[k]), device=DEV) for k in ("r", "beta", "beta_dot", "x_det", "charge")}
    E, diag = lw.deposit_td(t["r"], t["beta"], t["beta_dot"], c["t_start"], c["dt"], t["x_det"], c["t0"], c["dt_obs"],
                            c["n_obs"], prec=prec, field_mask=3, geom=geom, charge=t["charge"])
    Eo, do = oracle.deposit_td(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], c["dt_obs"],
                               c["n_obs"], charge=c["charge"], field_mask=3,
                               geom=oracle.GEOM_EXACT if geom == "exact" else oracle.GEOM_FARFIELD)
    assert diag.cpu().tolist() == list(do) and do[1] > 0
    assert np.max(np.abs(E.double().cpu().numpy() - Eo)) <= {"fp64": 1e-9, "mixed": 2e-5}[prec] * max(np.max(np.abs(Eo)), 1e-300)
