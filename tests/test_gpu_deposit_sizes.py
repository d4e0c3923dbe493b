"""lw_deposit_td of more short trajectories than one launch takes (2^23 particles; 2^26 / 128 = 2^19 of them with 128 tiles
of pixels): all but a few carry no charge, the others lie on both sides of the launches' ends, one of them on the careful
path.  Against the deposit of those few alone (order of the sums: 1e-12)."""
import numpy as np
import pytest
import torch

import oracle
from cases import synthetic

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n, at, n_pix, det", [((1 << 24) + 9, [0, (1 << 23) - 1, 1 << 23, (1 << 24) - 1, 1 << 24, (1 << 24) + 8], 3, False),
                                               ((1 << 23) + 9, [5, (1 << 23) - 1, 1 << 23, (1 << 23) + 8], 1, True),
                                               ((1 << 20) + 9, [5, (1 << 19) - 1, 1 << 19, (1 << 20) - 1, 1 << 20, (1 << 20) + 8], 16384, False)])
def test_many_short_trajectories(n, at, n_pix, det):
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=len(at), n_samples=2, n_pix=n_pix, n_obs=16)
    c["r"] = c["r"] - c["r"][:, :1]  # all start from one point: the window holds every one's interval
    tau, _, _ = oracle.eval_samples(0.0, c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"][:1], 0.0, 1.0)
    c["dt_obs"] = float(np.ptp(tau)) / 11
    c["t0"] = float(np.min(tau)) - 2 * c["dt_obs"]
    few = [torch.as_tensor(np.ascontiguousarray(c[k]), device=DEV) for k in ("r", "beta", "beta_dot")]
    few[1][1, 1, 0] = 1.5  # careful path: an unusable sample
    many = [f[:1].repeat(n, 1, 1) for f in few]
    for m, f in zip(many, few):
        m[torch.tensor(at, device=DEV)] = f
    q = torch.zeros(n, dtype=torch.float64, device=DEV)
    q[torch.tensor(at, device=DEV)] = torch.as_tensor(c["charge"], device=DEV)
    x = torch.as_tensor(np.ascontiguousarray(c["x_det"]), device=DEV)
    grid = (c["t_start"], c["dt"], x, c["t0"], c["dt_obs"], c["n_obs"])
    run = lw.deposit_td_det if det else (lambda *a, **k: lw.deposit_td(*a, prec="fp64", **k))
    E, d = run(*many, *grid, charge=q)
    Eo, do = run(*few, *grid, charge=torch.as_tensor(c["charge"], device=DEV))
    one = run(*[f[:1].contiguous() for f in few], *grid, charge=torch.as_tensor(c["charge"][:1], device=DEV))[1]
    assert float(Eo.abs().max()) > 0
    assert d.tolist() == [int(a) + (n - len(at)) * int(b) for a, b in zip(do.tolist(), one.tolist())]
    assert float((E - Eo).abs().max()) <= 1e-12 * float(Eo.abs().max())
