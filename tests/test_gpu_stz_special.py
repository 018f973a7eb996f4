"""GPU parity of the STZ step on values out of the ordinary: NaN and infinities
in the state, arguments of cosh up to where it overflows, and negative ones."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import stz as ostz
from workloads import lame, stz_constants

pytestmark = pytest.mark.gpu
LAM, MU = lame()
N = (12, 8, 6)


def dev(a):
    return torch.from_numpy(a.copy()).cuda()


def state(seed, load):
    nx, ny, nz = N
    rng = np.random.default_rng(seed)
    p = stz_constants()
    sigma = 0.05 * p["s_y"] * rng.standard_normal((6, nz, ny, nx))
    sigma[4] += load * p["s_y"]
    chi = 0.04 + 0.003 * rng.standard_normal((nz, ny, nx))
    return p, 1e-5 * rng.standard_normal((3, nz + 1, ny, nx)), sigma, chi


def step(p, dt, v, sigma, chi):
    from paper_1904_03808_amd.qsmg import MGSolver
    g = MGSolver(*N, 1.0 / N[2], LAM, MU, min_coarse_nz=3)
    ss, c1 = g.stz_step(p, dt, dev(v), dev(sigma), dev(chi))
    rs, rc = ostz.stz_step(v, sigma, chi, 1.0 / N[2], dt, LAM, MU, p)
    return ss.cpu().numpy(), c1.cpu().numpy(), rs, rc


@pytest.mark.parametrize("n_sub", [4, -1])
def test_nan_in_substeps(n_sub):
    """A NaN stress component makes the cell's chi NaN, a NaN chi leaves the
    cell's stress as the kinematic terms make it, and an infinite one is NaN from
    the first sub-step on, in cells above and below yield:
    NaN exactly where the oracle has it, other values to the bars of the STZ
    step's other parity cases."""
    p, v, sigma, chi = state(31, 1.1)
    sigma[:, :, 0] *= 0.5  # rows below yield
    sigma[0, 1, 2, 3] = sigma[4, 2, 3, 4] = sigma[1, 3, 0, 5] = np.nan
    chi[4, 0, 6] = np.nan
    chi[4, 0, 7] = np.inf
    if n_sub > 0:  # (per cell, a NaN chi above yield asks for the most sub-steps)
        chi[1, 5, 7] = chi[5, 7, 11] = np.nan
        chi[2, 5, 7] = np.inf
    with np.errstate(all="ignore"):
        ss, c1, rs, rc = step(dict(p, n_sub=n_sub), 10.0, v, sigma, chi)
    assert np.array_equal(np.isnan(c1), np.isnan(rc))
    assert np.array_equal(np.isnan(ss), np.isnan(rs))
    assert np.isnan(rc).sum() == (8 if n_sub > 0 else 5)
    largest = np.nan_to_num(np.abs(rs)).max(axis=0)  # of the cell (one overshoots far)
    assert np.all(np.nan_to_num(np.abs(ss - rs)) <= 1e-12 * largest)
    assert np.nanmax(np.abs(c1 - rc)) <= 1e-11 * np.abs(rc - chi)[np.isfinite(rc)].max() + 1e-16


@pytest.mark.parametrize("sign", [1, -1])
@pytest.mark.parametrize("n_sub", [1, -2])
def test_largest_arguments(sign, n_sub):
    """beta sbar between 709.8, where exp overflows, and 710.4, where cosh does not
    yet, and its negative.  The argument carries a few roundings (8 at most), which
    cosh multiplies by its size: 8 * 711 * 1.2e-16 of a cell's largest value."""
    p, v, sigma, chi = state(32, 0.0)
    sigma[4] = np.linspace(709.8, 710.4, sigma[4].size).reshape(sigma[4].shape) / p["beta"]
    sigma[[0, 1, 2, 3, 5]] = 0.0
    p = dict(p, n_sub=n_sub, beta=sign * p["beta"])
    # a step in which the plastic terms are of the order of the stress (the rate
    # is about 1e296), but for the implicit form, which takes any
    dt = 1e-297 if n_sub == 1 else 10.0
    ss, c1, rs, rc = step(p, dt, v, sigma, chi)
    assert np.isfinite(rs).all() and np.isfinite(rc).all()
    assert np.abs(rs - sigma).max() > 1e-3
    assert np.abs(ss - rs).max() <= 7e-13 * np.abs(rs).max()
    assert np.abs(c1 - rc).max() <= 7e-13 * np.abs(rc).max()


@pytest.mark.parametrize("n_sub", [1, 4, -1, -2])
def test_negative_beta(n_sub):
    """cosh is even: a negative beta at ordinary stresses, to the usual bars."""
    p, v, sigma, chi = state(33, 1.1)
    p = dict(p, n_sub=n_sub, beta=-p["beta"])
    ss, c1, rs, rc = step(p, 10.0, v, sigma, chi)
    assert np.abs(ss - rs).max() <= 1e-12 * np.abs(rs).max()
    assert np.abs(c1 - rc).max() <= 1e-11 * np.abs(rc - chi).max() + 1e-16


def test_negative_beta_far_from_zero():
    """Sub-steps at beta sbar about -420, where exp(-2 b) alone overflows; bars as
    for the largest arguments."""
    p, v, sigma, chi = state(34, 0.0)
    sigma[4] = np.linspace(415.0, 420.0, sigma[4].size).reshape(sigma[4].shape) / p["beta"]
    sigma[[0, 1, 2, 3, 5]] = 0.0
    chi[:] = 0.04
    D = ostz.plastic_rate(sigma[4].max(), 0.04, p)
    p = dict(p, n_sub=4, beta=-p["beta"])
    # the fastest cell loses 1e-4 of its stress (0.04 of the argument's unit)
    dt = 1e-4 * sigma[4].max() / (2 * MU * D)
    ss, c1, rs, rc = step(p, dt, v, sigma, chi)
    assert np.abs(rs - sigma).max() > 1e-5
    assert np.abs(ss - rs).max() <= 7e-13 * np.abs(rs).max()
    assert np.abs(c1 - rc).max() <= 7e-13 * np.abs(rc).max()
