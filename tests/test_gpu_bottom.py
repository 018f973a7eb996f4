"""GPU parity of the two coarsest levels applied as one map: coarsest sizes that
are odd, two or no power of two, other sweep counts and colour orders, and both
precisions.  (Where the map's blocks would be too large the levels run one by
one, as they do at every setup, whose responses the blocks are.)"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.multigrid import MGOracle
from workloads import lame

pytestmark = pytest.mark.gpu
LAM, MU = lame()
ROW, PLAIN = (0, 1, 4, 5, 2, 3, 6, 7), (0, 1, 2, 3, 4, 5, 6, 7)


# grid, min_coarse_nz, coarsest level
GRIDS = [((20, 28, 12), 3),   # 5 x 7 x 3
         ((8, 12, 8), 2),     # 2 x 3 x 2
         ((24, 8, 16), 4),    # 6 x 2 x 4
         ((32, 32, 32), 8),   # 8 x 8 x 8
         ((48, 40, 16), 2)]   # four levels to 6 x 5 x 2


@pytest.mark.parametrize("n,coarse", GRIDS)
@pytest.mark.parametrize("pre,post,order", [(2, 2, ROW), (1, 3, ROW), (2, 0, PLAIN)])
def test_cycles(n, coarse, pre, post, order):
    """Two FP64 V-cycles against the oracle, 1e-12 of the largest value (as for
    the V-cycle iterates where the levels run one by one)."""
    from paper_1904_03808_amd.qsmg import MGSolver
    nx, ny, nz = n
    g = MGSolver(nx, ny, nz, 1.0 / nz, LAM, MU, min_coarse_nz=coarse, n_pre=pre, n_post=post,
                 colour_order=order)
    o = MGOracle(nx, ny, nz, 1.0 / nz, LAM, MU, min_coarse_nz=coarse, n_pre=pre, n_post=post,
                 order=[(c & 1, (c >> 1) & 1, (c >> 2) & 1) for c in order])
    rng = np.random.default_rng(11)
    x = rng.standard_normal((3, nz + 1, ny, nx))
    b = rng.standard_normal((3, nz + 1, ny, nx)) * nz * nz
    b[:, 0] = b[:, -1] = 0
    xd = torch.from_numpy(x).cuda()
    g.solve(torch.from_numpy(b).cuda(), xd, rtol=1e-300, max_cycles=2, raise_on_failure=False)
    xr, _ = o.solve(b, x, rtol=1e-300, max_cycles=2)
    assert np.abs(xd.cpu().numpy() - xr).max() <= 1e-12 * np.abs(xr).max()


@pytest.mark.parametrize("n,coarse", [((20, 28, 12), 3), ((32, 32, 32), 8)])
def test_refinement(n, coarse):
    """FP32 cycles inside FP64 refinement reach 1e-10 by the oracle's residual
    in at most one cycle more than the FP64 solve takes."""
    from paper_1904_03808_amd.qsmg import MGSolver
    nx, ny, nz = n
    o = MGOracle(nx, ny, nz, 1.0 / nz, LAM, MU, min_coarse_nz=coarse)
    rng = np.random.default_rng(12)
    x = rng.standard_normal((3, nz + 1, ny, nx))
    b = rng.standard_normal((3, nz + 1, ny, nx)) * nz * nz
    b[:, 0] = b[:, -1] = 0
    cycles = []
    for precision in ("fp64", "fp32-ir"):
        g = MGSolver(nx, ny, nz, 1.0 / nz, LAM, MU, min_coarse_nz=coarse, precision=precision)
        xd = torch.from_numpy(x).cuda()
        cycles.append(g.solve(torch.from_numpy(b).cuda(), xd, rtol=1e-10).cycles)
        r = o.residual(xd.cpu().numpy(), b)
        assert np.linalg.norm(r) <= 1.01e-10 * o.lifted_rhs_norm(b, x)
    assert cycles[1] <= cycles[0] + 1
