"""GPU parity of the fine-level sweep by rows at every LDS row stride, also where
the size of the grid asks for tiles: rows that fill their stride and rows with
slack, workgroups of 1 to 37 rows of a parity with last groups that repeat a row,
and planes that leave a remainder."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.multigrid import MGOracle
from workloads import lame

pytestmark = pytest.mark.gpu
LAM, MU = lame()

# grid, min_coarse_nz: LDS stride; rows of one parity, R of them per workgroup
# (FP64, FP32)
GRIDS = [((16, 40, 8), 2),      # 36 with slack; 20 rows, R = 18 and 32
         ((32, 32, 32), 4),     # 36; 16 rows, R = 16
         ((8, 8, 16), 8),       # 36 with slack; 4 rows, R = 18 and 37
         ((16, 16, 64), 16),    # 36 with slack; 8 rows, R = 18 and 32
         ((34, 6, 10), 5),      # 52 with slack; 3 rows, R = 12 and 15
         ((40, 24, 32), 4),     # 52 with slack; 12 rows, R = 12
         ((64, 12, 8), 2),      # 68; 6 rows, R = 8
         ((66, 10, 6), 3),      # 84 with slack; 5 rows, R = 7
         ((84, 12, 8), 2),      # 100 with slack; 6 rows, R = 6
         ((98, 8, 6), 3),       # 132 with slack; 4 rows, R = 4 and 5
         ((128, 10, 8), 4),     # 132; 5 rows, R = 4
         ((136, 20, 12), 3),    # 164 with slack; 10 rows, R = 3
         ((170, 6, 6), 3),      # 196 with slack; 3 rows, R = 2 and 3
         ((192, 12, 20), 5),    # 196; 6 rows, R = 2
         ((200, 6, 6), 3),      # 260 with slack; 3 rows, R = 2
         ((300, 12, 12), 3),    # 324 with slack; R = 1 from here on
         ((320, 12, 8), 2),     # 324
         ((352, 12, 8), 2),     # 388 with slack
         ((386, 6, 4), 2)]      # 516 with slack, three planes


def solver(n, coarse, precision):
    from paper_1904_03808_amd.qsmg import MGSolver
    g = MGSolver(*n, 1.0 / n[2], LAM, MU, min_coarse_nz=coarse, precision=precision)
    g.fine_sweep_rows(True)
    return g, MGOracle(*n, 1.0 / n[2], LAM, MU, min_coarse_nz=coarse)


def fields(n, seed):
    nx, ny, nz = n
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((3, nz + 1, ny, nx))
    b = rng.standard_normal((3, nz + 1, ny, nx)) * nz * nz
    b[:, 0] = b[:, -1] = 0
    return x, b


@pytest.mark.parametrize("n,coarse", GRIDS)
def test_fp64(n, coarse):
    """One and three sweeps to 1e-13 of the largest value (sums of about 45 terms),
    walls untouched, and one V-cycle, whose first post-smoothing sweep adds the
    coarse correction as it reads, to 1e-12, the bars of the sweep and of the
    V-cycle iterates elsewhere."""
    g, o = solver(n, coarse, "fp64")
    x, b = fields(n, 3)
    for sweeps in (1, 3):
        xd = torch.from_numpy(x).cuda()
        g.smooth(0, xd, torch.from_numpy(b).cuda(), sweeps)
        xr = x.copy()
        for _ in range(sweeps):
            o.levels[0].sweep(xr, b, o.order)
        got = xd.cpu().numpy()
        assert np.abs(got - xr).max() <= 1e-13 * np.abs(xr).max(), sweeps
        assert np.array_equal(got[:, [0, -1]], x[:, [0, -1]])
    xd = torch.from_numpy(x).cuda()
    g.solve(torch.from_numpy(b).cuda(), xd, rtol=1e-300, max_cycles=1, raise_on_failure=False)
    xr, _ = o.solve(b, x, rtol=1e-300, max_cycles=1)
    assert np.abs(xd.cpu().numpy() - xr).max() <= 1e-12 * np.abs(xr).max()


@pytest.mark.parametrize("n,coarse", GRIDS)
def test_fp32(n, coarse):
    """One and three sweeps to 2e-6 of the largest value on the same rounded inputs,
    and a solve, whose cycles start from a zero correction that is not read and add
    the coarse correction as they read: 1e-10 by the oracle's residual in at most
    two cycles more than the oracle's FP64 ones."""
    g, o = solver(n, coarse, "fp32-ir")
    x, b = fields(n, 4)
    xf, bf = x.astype(np.float32), b.astype(np.float32)
    for sweeps in (1, 3):
        xd = torch.from_numpy(xf).cuda()
        g.smooth(0, xd, torch.from_numpy(bf).cuda(), sweeps)
        xr = xf.astype(np.float64)
        for _ in range(sweeps):
            o.levels[0].sweep(xr, bf.astype(np.float64), o.order)
        got = xd.cpu().numpy()
        assert np.abs(got - xr).max() <= 2e-6 * np.abs(xr).max(), sweeps
        assert np.array_equal(got[:, [0, -1]], xf[:, [0, -1]])
    xd = torch.from_numpy(x).cuda()
    info = g.solve(torch.from_numpy(b).cuda(), xd, rtol=1e-10)
    r = o.residual(xd.cpu().numpy(), b)
    assert np.linalg.norm(r) <= 1.01e-10 * o.lifted_rhs_norm(b, x)
    _, oi = o.solve(b, x, rtol=1e-10)
    assert info.cycles <= oi["cycles"] + 2


def test_rows_and_tiles_agree():
    """Both kernels on one handle, switched back and forth, and a value that is
    neither is refused."""
    n = (34, 6, 10)
    g, _ = solver(n, 5, "fp64")
    x, b = fields(n, 5)
    out = []
    for rows in (True, False, True):
        g.fine_sweep_rows(rows)
        xd = torch.from_numpy(x).cuda()
        g.smooth(0, xd, torch.from_numpy(b).cuda(), 2)
        out.append(xd.cpu().numpy())
    assert np.array_equal(out[0], out[2])
    assert np.abs(out[0] - out[1]).max() <= 1e-13 * np.abs(out[0]).max()
    assert g._lib.qs_fine_sweep_rows(g._h, 2) == -1
