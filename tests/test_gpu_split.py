"""GPU parity where the work of a launch is split by size: the segment lengths
of the fine residual and the fused residual and restriction, at grids whose
planes leave a remainder for each of them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.multigrid import MGOracle
from workloads import lame

pytestmark = pytest.mark.gpu
LAM, MU = lame()


def pair(nx, ny, nz, coarse, n_pre=2, n_post=2, precision="fp64"):
    from paper_1904_03808_amd.qsmg import MGSolver
    order = (0, 1, 4, 5, 2, 3, 6, 7)
    g = MGSolver(nx, ny, nz, 1.0 / nz, LAM, MU, min_coarse_nz=coarse, n_pre=n_pre, n_post=n_post,
                 precision=precision, colour_order=order)
    o = MGOracle(nx, ny, nz, 1.0 / nz, LAM, MU, min_coarse_nz=coarse, n_pre=n_pre, n_post=n_post,
                 order=[(c & 1, (c >> 1) & 1, (c >> 2) & 1) for c in order])
    return g, o


def fields(nx, ny, nz, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((3, nz + 1, ny, nx))
    b = rng.standard_normal((3, nz + 1, ny, nx)) * nz * nz
    b[:, 0] = b[:, -1] = 0
    return x, b


# residual segments of 2 planes with one left over and of 4 with three (96^3),
# restriction segments of 1 and of 2 coarse planes (96^3), ragged tiles, and a
# single interior coarse plane
@pytest.mark.parametrize("n,coarse", [((6, 6, 4), 2), ((66, 10, 6), 3), ((96, 32, 12), 3),
                                      ((96, 96, 96), 6)])
def test_one_cycle_with_short_segments(n, coarse):
    """One FP64 V-cycle from a random start with wall data, and the norm of its
    residual, against the oracle: 1e-12 of the largest value, as for the
    V-cycle iterates elsewhere (a cycle is a few dozen sums of about 100 terms)."""
    g, o = pair(*n, coarse)
    x, b = fields(*n, 7)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(b).cuda()
    info = g.solve(bd, xd, rtol=1e-300, max_cycles=1, raise_on_failure=False)
    xr, oi = o.solve(b, x, rtol=1e-300, max_cycles=1)
    assert np.abs(xd.cpu().numpy() - xr).max() <= 1e-12 * np.abs(xr).max()
    assert np.allclose(info.hist, oi["hist"][:2], rtol=1e-11, atol=0)
