"""The pusher at the edges of its blocks (32 particles with two lanes each, or 64 with one beyond 32768
particles) and of its hand-over batches (8 or 4 samples), against the oracle with the tolerances of
test_gpu_fft_fd_boris.py (1e-12 of the positions and of beta, 1e-9 of beta_dot); a particle's samples
are the same bits whichever layout pushes it."""
import numpy as np
import pytest
import torch

import oracle
from paper_2206_03015_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def setup(n_p, n_samples, w0):
    W = inputs.workload("bunch").scaled(n_p=n_p, n_steps=600)
    init = inputs.bunch_init(W)
    # start inside the pulse, so that every sample of a short push sees the field
    init[:, 2] = np.random.default_rng(n_p).uniform(-2e-6, 2e-6, n_p)
    L = W.laser
    return init, (n_samples, -1e-15, W.dt, L.a0, L.lam, w0, L.n_cycles)


@pytest.mark.parametrize("w0", [10e-6, 0.0])
@pytest.mark.parametrize("n_p, n_samples", [(1, 1), (1, 600), (31, 2), (32, 7), (33, 8), (64, 9), (65, 17), (300, 33)])
def test_push_edges(n_p, n_samples, w0):
    from paper_2206_03015_amd import lw
    init, args = setup(n_p, n_samples, w0)
    ns, t_start, dt, a0, lam, w0, nc = args
    ref = oracle.boris(init, ns, t_start, dt, a0, lam, w0, nc)
    got = [x.cpu().numpy() for x in lw.trajectory_boris(torch.as_tensor(init, device=DEV), *args)]
    for g, o, tol in zip(got, ref, (1e-12, 1e-12, 1e-9)):
        assert g.shape == o.shape == (n_p, n_samples, 3)
        assert np.max(np.abs(g - o)) <= tol * np.max(np.abs(o))


@pytest.mark.parametrize("n_samples", [1, 3, 4, 5, 21])
def test_layouts_give_the_same_bits(n_samples):
    from paper_2206_03015_amd import lw
    init, args = setup(32768 + 70, n_samples, 10e-6)
    it = torch.as_tensor(init, device=DEV)
    whole = lw.trajectory_boris(it, *args)
    for lo, hi in ((0, 100), (32700, 32768 + 70)):
        part = lw.trajectory_boris(it[lo:hi].contiguous(), *args)
        for a, b in zip(whole, part):
            assert torch.equal(a[lo:hi], b)
