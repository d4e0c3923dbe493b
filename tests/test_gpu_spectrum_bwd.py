"""lw_spectrum_fft_bwd in single precision on the workloads' own grid steps, whose factor dt_obs^2 / pi lies below the
smallest normal float, for dS down to where the gradient itself would leave the normal range.  Against the formula in
FP64; bound 1e-5 of the largest element (some 40 radix and twiddle roundings of 2^-24 in a transform and
its inverse, in random directions: a few 1e-7)."""
import numpy as np
import pytest
import torch

from oracle import gradient as og
from paper_2206_03015_amd import inputs

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


# 2^10 and 2^12 points take the runtime-shaped passes, the others the compile-time ones
@pytest.mark.parametrize("name, size, n_obs", [("bunch", 1.0, 1 << 18), ("bunch", 1e-4, 1 << 18), ("bunch", 1e-8, 1 << 18),
                                               ("bunch", 1.0, 1 << 10), ("bunch", 1e-4, 1 << 14),
                                               ("precision", 1.0, 1 << 18), ("precision", 1e-4, 1 << 18),
                                               ("precision", 1.0, 1 << 12), ("precision", 1.0, 1 << 13)])
def test_mixed_adjoint_at_the_workloads_grid_steps(name, size, n_obs):
    from paper_2206_03015_amd import lw
    dt = inputs.workload(name).dt_obs
    rng = np.random.default_rng(n_obs)
    E = torch.as_tensor(rng.normal(size=(3, 3, n_obs)) * 1e5, dtype=torch.float32)
    dS = torch.as_tensor(rng.normal(size=(3, n_obs // 2 + 1)) * size, dtype=torch.float32)
    ref = og.spectrum_vjp(E.double().numpy(), dS.double().numpy(), dt)
    assert np.max(np.abs(ref)) > 4 * np.finfo(np.float32).tiny
    dE = lw.spectrum_fft_bwd(E.to(DEV), dS.to(DEV), dt, "mixed").double().cpu().numpy()
    err = np.max(np.abs(dE - ref)) / np.max(np.abs(ref))
    print(f"{name} dS {size:g} n_obs {n_obs}: rel err {err:.2e}")
    assert err <= 1e-5
