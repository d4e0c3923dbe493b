"""Which frequency lists the FP64 direct sum takes as equally spaced, and lists of every length of its tiles."""
import numpy as np
import pytest
import torch

import oracle
from cases import synthetic

pytestmark = pytest.mark.gpu
DEV = "cuda"


def T(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


def args(c, omega):
    return (T(c["r"]), T(c["beta"]), T(c["beta_dot"]), c["t_start"], c["dt"], T(c["x_det"]), c["t0"], T(omega))


@pytest.mark.parametrize("off, taken", [(0.0, True), (2.0, True), (6.0, False), (8.0, False)])
def test_lists_at_the_tolerance(off, taken):
    """Every second frequency `off` x 2^-53 of itself above the line.  A list that is not taken as equally spaced is summed
    frequency by frequency, with the bits of the same list in another order; the line's sums have other bits.  (One
    chunk of samples, so that nothing is added in another order.)  Both within 1e-10 (the phase is below 2 pi 1e4,
    6.3e4 x 4 x 1.1e-16 = 2.8e-11 of a term, twice that in a square)."""
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=1, n_samples=200, n_pix=3)
    n = 64
    w = np.linspace(1e18, 2e18, n, dtype=np.longdouble)
    w[::2] *= 1 + np.longdouble(off) * np.longdouble(2.0) ** -53
    w = w.astype(np.float64)
    perm = np.random.default_rng(3).permutation(n)
    S = lw.direct_fd(*args(c, w), prec="fp64").cpu().numpy()
    P = lw.direct_fd(*args(c, w[perm]), prec="fp64").cpu().numpy()
    assert np.array_equal(S[:, perm], P) != taken
    So = oracle.direct_fd(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], w)
    assert np.max(np.abs(S - So)) <= 1e-10 * So.max() and np.max(np.abs(P - So[:, perm])) <= 1e-10 * So.max()
