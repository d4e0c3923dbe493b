"""The FP64 direct sum and its adjoint where the frequencies are equally spaced (sums as matrix products over blocks
of 32 frequencies) and where they are not (one sine/cosine pair per term), at the edges of blocks and tiles."""
import numpy as np
import pytest
import torch

import oracle
from cases import synthetic

pytestmark = pytest.mark.gpu
DEV = "cuda"
# The phase w t of these cases is below 2 pi 1e4, so its rounding moves a term by at most 2 pi 1e4 x 2 x 1.1e-16
# = 1.4e-11 of itself; bound of a spectrum or gradient against its largest element or its norm: 1e-10.
TOL = 1e-10


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


def args(c, omega):
    return (T(c["r"]), T(c["beta"]), T(c["beta_dot"]), c["t_start"], c["dt"], T(c["x_det"]), c["t0"], T(omega))


@pytest.mark.parametrize("geom", ["exact", "farfield"])
@pytest.mark.parametrize("n_w,n_samples", [(2, 5), (31, 64), (33, 257), (256, 31), (257, 300), (513, 70), (1030, 513)])
def test_equal_spacing_against_oracle_and_permuted_list(geom, n_w, n_samples):
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=3, n_samples=n_samples, n_pix=5)
    omega = np.linspace(1e18, 2e19, n_w)
    perm = np.random.default_rng(n_w).permutation(n_w)
    So = oracle.direct_fd(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], omega,
                          charge=c["charge"], geom=oracle.GEOM_FARFIELD if geom == "farfield" else oracle.GEOM_EXACT)
    dS = np.random.default_rng(1).random(So.shape) / So.max()
    out = {}
    for name, p in (("equal", np.arange(n_w)), ("permuted", perm)):
        S = lw.direct_fd(*args(c, omega[p]), prec="fp64", geom=geom, charge=T(c["charge"])).cpu().numpy()
        err = np.max(np.abs(S - So[:, p])) / So.max()
        print(f"{geom} {name} {n_w} frequencies, {n_samples} samples: {err:.2e}")
        assert err <= TOL
        out[name] = lw.direct_fd_bwd(*args(c, omega[p]), T(dS[:, p]), geom=geom, charge=T(c["charge"]))
    for a, b, what in zip(out["equal"], out["permuted"], ("r", "beta", "beta_dot")):
        err = float(torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b))
        print(f"{geom} d{what}: {err:.2e}")
        assert err <= TOL


def test_list_that_starts_at_zero_and_descending_list():
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=2, n_samples=200, n_pix=2)
    for omega in (np.linspace(0.0, 2e19, 65), np.linspace(2e19, 1e18, 100)):
        So = oracle.direct_fd(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], omega,
                              charge=c["charge"])
        S = lw.direct_fd(*args(c, omega), prec="fp64", charge=T(c["charge"])).cpu().numpy()
        assert np.max(np.abs(S - So)) / So.max() <= TOL
