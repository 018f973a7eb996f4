"""GPU parity of the STZ step and the explicit step where their work is split or
rearranged: bands of 16 rows cut into segments of planes for the eight XCDs (9
bands, planes that leave a remainder), sub-steps that overshoot, and the wall
planes of the explicit step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import stz as ostz
from workloads import lame, stz_constants

pytestmark = pytest.mark.gpu
LAM, MU = lame()


def state(n, seed, load):
    nx, ny, nz = n
    rng = np.random.default_rng(seed)
    p = stz_constants()
    sigma = 0.05 * p["s_y"] * rng.standard_normal((6, nz, ny, nx))
    sigma[4] += load * p["s_y"]
    chi = 0.04 + 0.003 * rng.standard_normal((nz, ny, nx))
    v = 1e-5 * rng.standard_normal((3, nz + 1, ny, nx))
    return p, v, sigma, chi


def handle(n, coarse):
    from paper_1904_03808_amd.qsmg import MGSolver
    return MGSolver(*n, 1.0 / n[2], LAM, MU, min_coarse_nz=coarse)


def dev(a):
    return torch.from_numpy(a.copy()).cuda()


# 9 bands of rows (segments of 2 planes, five whole and one of one), 1 band with
# fewer planes than XCDs, a ragged band
@pytest.mark.parametrize("n,coarse", [((20, 136, 12), 3), ((20, 16, 4), 2), ((24, 40, 12), 3)])
@pytest.mark.parametrize("opts", [dict(advect=1), dict(advect=1, l_diff=0.1, n_sub=-1)])
def test_advected_step(n, coarse, opts):
    """sigma* to 1e-12 of its largest value and the chi increment to 1e-11, the
    bars of the STZ step's other parity cases."""
    p, v, sigma, chi = state(n, 21, 1.05)
    p = dict(p, **opts)
    g = handle(n, coarse)
    ss, c1 = g.stz_step(p, 10.0, dev(v), dev(sigma), dev(chi))
    rs, rc = ostz.stz_step(v, sigma, chi, 1.0 / n[2], 10.0, LAM, MU, p)
    assert np.abs(ss.cpu().numpy() - rs).max() <= 1e-12 * np.abs(rs).max()
    assert np.abs(c1.cpu().numpy() - rc).max() <= 1e-11 * np.abs(rc - chi).max() + 1e-16


@pytest.mark.parametrize("dt", [200.0, 2e3, 2e4])
def test_fixed_substeps(dt):
    """Four sub-steps whatever the state: with dt = 2e3 and 2e4 some cells take
    more than their whole deviator off in one (it changes sign, and stops where it
    ends below yield).  Bars as above; the increments of cells past one overshoot
    are of the order of the stress itself."""
    n = (12, 8, 6)
    p, v, sigma, chi = state(n, 22, 1.1)
    p = dict(p, n_sub=4)
    g = handle(n, 3)
    ss, c1 = g.stz_step(p, dt, dev(v), dev(sigma), dev(chi))
    rs, rc = ostz.stz_step(v, sigma, chi, 1.0 / n[2], dt, LAM, MU, p)
    ok = np.isfinite(rs).all(axis=0) & (np.abs(rs).max(axis=0) < 1.0)
    assert ok.mean() > 0.5
    assert np.abs(ss.cpu().numpy() - rs)[:, ok].max() <= 1e-12 * np.abs(rs[:, ok]).max()
    assert np.abs(c1.cpu().numpy() - rc)[ok].max() <= 1e-11 * np.abs(rc - chi)[ok].max()


@pytest.mark.parametrize("n,coarse", [((20, 136, 12), 3), ((6, 4, 2), 2)])
def test_explicit_step(n, coarse):
    """Two explicit steps: v and sigma to 1e-12, chi to 1e-14, walls exactly."""
    p, v, sigma, chi = state(n, 23, 1.02)
    h = 1.0 / n[2]
    g = handle(n, coarse)
    vd, sd, cd = dev(v), dev(sigma), dev(chi)
    dt = h * h / 20
    for _ in range(2):
        g.explicit_step(p, dt, 1e-3, MU, 4.8 * h, vd, sd, cd)
        v, sigma, chi = ostz.explicit_step(v, sigma, chi, h, dt, LAM, MU, p, 1e-3, MU, 4.8 * h)
    assert np.abs(vd.cpu().numpy() - v).max() <= 1e-12 * np.abs(v).max()
    assert np.abs(sd.cpu().numpy() - sigma).max() <= 1e-12 * np.abs(sigma).max()
    assert np.abs(cd.cpu().numpy() - chi).max() <= 1e-14
    assert np.array_equal(vd.cpu().numpy()[:, [0, -1]], v[:, [0, -1]])
