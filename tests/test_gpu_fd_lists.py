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


@pytest.mark.parametrize("n_w", [1, 3, 64, 65, 100, 192, 193, 257, 300, 513, 1030])
@pytest.mark.parametrize("n_samples", [1, 5, 66, 300])
def test_uneven_lists_of_any_length(n_w, n_samples):
    """A sine/cosine pair per term (the order of a list does not matter to it): ends of the groups of 64 and 256
    frequencies, of a chunk of samples and of its quarters.  Tolerance as above."""
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=3, n_samples=n_samples, n_pix=2)
    w = np.geomspace(1e18, 2e19, n_w)
    w[:: 2] *= 1.0 + 1e-6
    S = lw.direct_fd(*args(c, w), prec="fp64", charge=T(c["charge"])).cpu().numpy()
    So = oracle.direct_fd(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], w, charge=c["charge"])
    assert np.max(np.abs(S - So)) <= 1e-10 * So.max()


@pytest.mark.parametrize("n_p, n_samples", [(600, 1), (300, 3), (257, 61), (256, 128), (256, 129)])
@pytest.mark.parametrize("spacing", ["equal", "uneven"])
def test_many_short_trajectories(n_p, n_samples, spacing):
    """At most half a chunk of samples each, from 512 blocks on: the chunks hold several particles (129: one each).  With a
    charge of its own per particle and an unusable sample.  Tolerance as above."""
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=n_p, n_samples=n_samples, n_pix=2)
    c["beta"][n_p // 2, n_samples // 2, 1] = np.nan
    w = (np.linspace if spacing == "equal" else np.geomspace)(1e18, 2e19, 70)
    S = lw.direct_fd(*args(c, w), prec="fp64", charge=T(c["charge"])).cpu().numpy()
    So = oracle.direct_fd(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], w, charge=c["charge"])
    assert np.max(np.abs(S - So)) <= 1e-10 * So.max()


@pytest.mark.parametrize("n_w, spacing", [(150, "equal"), (150, "uneven"), (4200, "equal")])
@pytest.mark.parametrize("n_p, n_samples, n_pix", [(1, 200, 13), (3, 70, 5), (2, 64, 4)])
def test_adjoint_adds_in_order(n_p, n_samples, n_pix, n_w, spacing):
    """The adjoint with the least workspace (a block takes all pixels) and with room for shares of them, repeated on sums of
    one chunk (n_p = 1, no atomics that meet): the same bits each time; both against each other and added to what
    is there.  4200 frequencies: more blocks of them than keep their centres in LDS."""
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=n_p, n_samples=n_samples, n_pix=n_pix)
    w = (np.linspace if spacing == "equal" else np.geomspace)(1e18, 2e19, n_w)
    dS = T(np.random.default_rng(2).random((n_pix, n_w)) * 1e30)
    least = lw.workspace_bytes(lw.WS_DIRECT_FD_BWD, n_pix, n_w, "fp64")
    out = {}
    for extra in (0, 2 * 72 * n_p * n_samples + 8, None):
        ws = None if extra is None else torch.empty((least + extra + 255) // 256 * 256, dtype=torch.uint8, device=DEV)[:least + extra]
        for rep in range(8 if n_p == 1 else 1):
            g = lw.direct_fd_bwd(*args(c, w), dS, ws=ws)
            if rep:
                assert all(torch.equal(a, b) for a, b in zip(g, out[extra]))
            out[extra] = g
    for a, b, d in zip(out[0], out[None], out[2 * 72 * n_p * n_samples + 8]):
        assert float(a.abs().max()) > 0
        assert float((a - b).abs().max()) <= 1e-12 * float(a.abs().max())
        assert float((a - d).abs().max()) <= 1e-12 * float(a.abs().max())
    twice = lw.direct_fd_bwd(*args(c, w), dS, out=tuple(a.clone() for a in out[None]))
    for a, b in zip(twice, out[None]):
        assert float((a - 2 * b).abs().max()) <= 1e-12 * float(b.abs().max())


@pytest.mark.parametrize("n_w, layout", [(1537, "equal"), (2048, "equal"), (2048, "piecewise"), (2048, "uneven"), (4097, "equal"),
                                         (4097, "piecewise")])
@pytest.mark.parametrize("n_samples", [5, 257, 300])
def test_mixed_sums_with_four_wavefronts_to_a_block(n_w, layout, n_samples):
    """From 1537 frequencies on (four wavefronts of 512, or nine: the last block's second to fourth have none and only stage
    samples) 256 samples are staged once for the block's wavefronts.  "piecewise" changes its spacing inside the third
    wavefront, which takes a sine/cosine pair per phasor beside the others' recurrence.  Tolerance of the mixed sums:
    1e-4 of the largest."""
    from paper_2206_03015_amd import lw
    c = synthetic(n_p=2, n_samples=n_samples, n_pix=3)
    w = np.linspace(1e17, 2e19, n_w)
    if layout == "piecewise":
        w[1300:] = w[1300] + 1.3 * (w[1300:] - w[1300])
    elif layout == "uneven":
        w = np.sort(np.random.default_rng(5).uniform(1e17, 2e19, n_w))
    S = lw.direct_fd(*args(c, w), prec="mixed", charge=T(c["charge"])).cpu().numpy()
    So = oracle.direct_fd(c["t_start"], c["dt"], c["r"], c["beta"], c["beta_dot"], c["x_det"], c["t0"], w, charge=c["charge"])
    err = np.max(np.abs(S - So)) / So.max()
    print(f"mixed, {n_w} {layout} frequencies, {n_samples} samples: rel err {err:.2e}")
    assert err <= 1e-4
