"""The direct sum and its adjoint beyond one launch: more pixels, resp. more short trajectories, than a grid of
256-thread blocks holds (2^24).  Compared with the same call on the few whose result is looked at: the same terms
in the same order."""
import numpy as np
import pytest
import torch

from cases import synthetic

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_many_pixels(prec):
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=1, n_samples=2, n_pix=7)
    n = (1 << 24) + 3
    x = T(c["x_det"]).repeat((n + 6) // 7, 1)[:n].contiguous()
    args = (T(c["r"]), T(c["beta"]), T(c["beta_dot"]), c["t_start"], c["dt"])
    omega = T(np.array([3e18]))
    S = lw.direct_fd(*args, x, c["t0"], omega, prec=prec)
    few = lw.direct_fd(*args, x[:7].contiguous(), c["t0"], omega, prec=prec)
    assert float(few.min()) > 0
    want = few.repeat((n + 6) // 7, 1)[:n]
    assert float(((S - want) / want).abs().max()) <= 1e-12


def test_adjoint_of_many_short_trajectories():
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=5, n_samples=2, n_pix=1)
    n = (1 << 24) + 4
    many = [T(c[k]).repeat((n + 4) // 5, 1, 1)[:n].contiguous() for k in ("r", "beta", "beta_dot")]
    # one particle of each kind carries a charge: the sums are those of the five
    q = torch.zeros(n, dtype=torch.float64, device=DEV)
    at = torch.tensor([0, 6, 4096 + 1, (1 << 24) + 2, (1 << 23) + 1], device=DEV)
    at = at - (at % 5) + torch.arange(5, device=DEV)
    at = torch.where(at >= n, at - 5, at)
    q[at] = T(c["charge"])
    omega, dS = T(np.array([3e18, 5e18])), T(np.array([[1.0, 2.0]]))
    x = T(c["x_det"])
    got = lw.direct_fd_bwd(*many, c["t_start"], c["dt"], x, c["t0"], omega, dS, charge=q)
    want = lw.direct_fd_bwd(*[T(c[k]) for k in ("r", "beta", "beta_dot")], c["t_start"], c["dt"], x, c["t0"], omega, dS,
                            charge=T(c["charge"]))
    for g, w in zip(got, want):
        assert float(w.abs().max()) > 0
        assert float((g[at] - w).abs().max()) <= 1e-10 * float(w.abs().max())
        assert float(g.abs().sum()) <= (1 + 1e-9) * float(w.abs().sum())
