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


# the larger of these take the compile-time passes, the others the runtime-shaped ones
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


# (pixels on both sides of the line between the runtime-shaped and the compile-time passes, odd ones among them)
@pytest.mark.parametrize("prec, lg, n_pix", [("mixed", 13, 62), ("mixed", 13, 63), ("mixed", 14, 64), ("mixed", 14, 67), ("mixed", 15, 33),
                                             ("mixed", 16, 16), ("mixed", 16, 17), ("mixed", 17, 6), ("mixed", 17, 7), ("mixed", 18, 1),
                                             ("fp64", 12, 62), ("fp64", 12, 63), ("fp64", 13, 64), ("fp64", 13, 65), ("fp64", 14, 35),
                                             ("fp64", 15, 16), ("fp64", 15, 17), ("fp64", 16, 6), ("fp64", 16, 7), ("fp64", 17, 1),
                                             ("fp64", 17, 2)])
def test_adjoint_on_both_sides_of_the_few_pixels_line(prec, lg, n_pix):
    """Against the formula in FP64; bounds 1e-5 as above and 1e-14 (the same roundings of 2^-53)."""
    from paper_2206_03015_amd import lw
    n_obs, dtype = 1 << lg, torch.float64 if prec == "fp64" else torch.float32
    rng = np.random.default_rng(lg + n_pix)
    E = torch.as_tensor(rng.normal(size=(n_pix, 3, n_obs)) * 1e5, dtype=dtype)
    dS = torch.as_tensor(rng.normal(size=(n_pix, n_obs // 2 + 1)), dtype=dtype)
    ref = og.spectrum_vjp(E.double().numpy(), dS.double().numpy(), 4.7e-20)
    dE = lw.spectrum_fft_bwd(E.to(DEV), dS.to(DEV), 4.7e-20, prec).double().cpu().numpy()
    err = np.max(np.abs(dE - ref)) / np.max(np.abs(ref))
    print(f"{prec} 2^{lg}, {n_pix} pixels: rel err {err:.2e}")
    assert err <= (1e-14 if prec == "fp64" else 1e-5)


@pytest.mark.parametrize("prec, lg, n_pix, bound", [("fp64", 16, 16, 4.7e-16), ("fp64", 19, 3, 5.0e-16), ("mixed", 16, 64, 2.8e-7),
                                                    ("mixed", 18, 16, 2.9e-7)])
def test_adjoint_is_as_accurate_as_tables_of_all_twiddles(prec, lg, n_pix, bound):
    """Root mean square error of the compile-time passes against the formula in long double, relative to the gradient's.
    Passes whose twiddles are all rounded once have 3.7e-16 (2^16) and 4.0e-16 (2^19) in FP64, 2.15e-7 and
    2.25e-7 in single precision; the bounds leave a quarter to the order of the radices.  Product chains of twiddles have
    6.1e-16, 6.7e-16, 5.3e-7 and 5.6e-7."""
    from paper_2206_03015_amd import lw
    n, dtype = 1 << lg, torch.float64 if prec == "fp64" else torch.float32
    rng = np.random.default_rng(lg)
    E = torch.as_tensor(rng.normal(size=(n_pix, 3, n)) * 1e5, dtype=dtype)
    dS = torch.as_tensor(rng.normal(size=(n_pix, n // 2 + 1)), dtype=dtype)
    dt = 2e-19
    got = lw.spectrum_fft_bwd(E.to(DEV), dS.to(DEV), dt, prec).double().cpu().numpy()
    wide = np.longdouble if prec == "fp64" else np.float64
    F = np.fft.rfft(E.numpy().astype(wide), axis=-1) * dS.numpy().astype(wide)[:, None]
    F[..., 1:-1] *= wide(0.5)
    ref = np.fft.irfft(F, n=n, axis=-1) * (n * wide(dt) * wide(dt) / wide("3.14159265358979323846264338327950288"))
    err = float(np.sqrt(np.mean((got - ref) ** 2) / np.mean(ref ** 2)))
    print(f"{prec} 2^{lg}: rms error {err:.2e}")
    assert err <= bound
