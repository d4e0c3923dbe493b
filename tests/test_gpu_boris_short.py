"""Short pushed trajectories and spans of 1500 particles and more, whose arrival bases and flags the pusher leaves: as the
deposit of the stored samples.  Tolerances as in test_gpu_boris_stream.py (the order of the sums alone differs)."""
import numpy as np
import pytest
import torch

from paper_2206_03015_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n_p, n_samples, span, prec", [(1499, 2, 0, "fp64"), (1500, 1, 0, "fp64"), (1500, 2, 0, "mixed"), (2100, 7, 0, "fp64"), (2100, 9, 2, "fp64"),
                                                        (2079, 301, 0, "mixed"), (2100, 1025, 9, "fp64"), (2100, 3001, 1000, "mixed"),
                                                        (32768 + 40, 6, 0, "fp64")])
def test_short_spans(n_p, n_samples, span, prec):
    from paper_2206_03015_amd import lw
    W = inputs.workload("bunch").scaled(n_p=n_p, n_steps=n_samples - 1 if n_samples > 1 else 1, n_side=3, n_obs=1 << 14)
    L = W.laser
    i0 = inputs.bunch_init(W)
    i0[:, 2] = np.random.default_rng(n_p).uniform(-2e-8, 2e-8, n_p)
    i0[1, 5] = 1e7
    i0[2, 4] = np.nan
    dt = 0.02 * L.lam / inputs.C_LIGHT
    init = torch.as_tensor(i0, device=DEV)
    x_det = torch.as_tensor(inputs.pixel_positions(W.n_side, W.theta_max, W.D), device=DEV)
    args = (n_samples, -0.3 * n_samples * dt, dt, L.a0, L.lam, L.w0, L.n_cycles)
    t0 = args[1] - 3e-16
    # points per sample interval 0.5, over the particles' offsets and the trajectory
    dt_obs = max(dt * n_samples / (2 * W.gamma ** 2), 2e-16) * 4 / W.n_obs
    grid = (x_det, t0, dt_obs, W.n_obs)
    Es, ds = lw.deposit_td_boris(init, *args, *grid, prec=prec, span=span)
    r, b, bd = lw.trajectory_boris(init, *args)
    Eo, do = lw.deposit_td(r, b, bd, args[1], dt, *grid, prec=prec)
    assert ds.tolist() == do.tolist() and (int(do[3]) > 0 or n_samples == 1)
    assert float((Es - Eo).abs().max()) <= (1e-12 if prec == "fp64" else 1e-6) * float(Eo.abs().max())
