"""GPU parity of the residual and its restriction as the V-cycle forms them, in
both working precisions, at sampled coarse nodes: each is evaluated by the oracle
on the 5 x 5 x 5 nodes around it, so that the size of the grid does not matter."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.multigrid import Level, fine_stencil, galerkin_stencil, restrict
from workloads import lame

LAM, MU = lame()


def check(n, coarse, level, precision, samples=400):
    """Values to 144 roundings of half a unit (27 residuals of about 45 terms each,
    whose largest partial sums may be twice the largest result)."""
    from paper_1904_03808_amd.qsmg import MGSolver
    g = MGSolver(*n, 1.0 / n[2], LAM, MU, min_coarse_nz=coarse, precision=precision)
    nx, ny, nz = g.level_dims(level)
    A = fine_stencil(n[2], 1.0 / n[2], LAM, MU)
    for l in range(level):
        A = galerkin_stencil(A, n[2] >> l)
    dt = torch.float32 if precision == "fp32-ir" else torch.float64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    x = torch.randn((3, nz + 1, ny, nx), generator=gen, device="cuda", dtype=dt)
    b = torch.randn((3, nz + 1, ny, nx), generator=gen, device="cuda", dtype=dt) * (nz * nz)
    bc = g.level_residual_restrict(level, x, b)
    torch.cuda.synchronize()
    assert not bc[:, [0, -1]].any()
    assert (bc[:, 1:-1] != 0).any(dim=0).all()  # no node left out
    rng = np.random.default_rng(8)
    K = rng.integers(1, nz // 2, samples)
    K[:40], K[40:80] = 1, nz // 2 - 1
    J, I = rng.integers(0, ny // 2, samples), rng.integers(0, nx // 2, samples)
    J[:100:2], I[1:100:2] = 0, 0
    J[100:140], I[120:160] = ny // 2 - 1, nx // 2 - 1
    # with the few nodes where a component happens to be zero
    zero = torch.nonzero((bc[:, 1:-1] == 0).any(dim=0))[:40].cpu().numpy()
    K, J, I = (np.concatenate([a, z]) for a, z in zip((K, J, I), (zero[:, 0] + 1, zero[:, 1], zero[:, 2])))
    at = torch.arange(-2, 3)
    got = bc[:, K, J, I].double().cpu().numpy()
    want = np.empty_like(got)
    for s in range(len(K)):
        ks, js, is_ = 2 * K[s] + at, (2 * J[s] + at) % ny, (2 * I[s] + at) % nx
        cut = lambda f: f[:, ks][:, :, js][..., is_].double().cpu().numpy()  # noqa: E731
        r = cut(b) - Level(5, 5, 4, A[2 * K[s] - 2:2 * K[s] + 3]).apply(cut(x))
        w = np.array([0.5, 1.0, 0.5])
        want[:, s] = np.einsum("cxyz,x,y,z->c", r[:, 1:4, 1:4, 1:4], w, w, w)
    assert np.abs(got - want).max() <= 72 * torch.finfo(dt).eps * np.abs(want).max()


def test_evaluation_by_nodes():
    """The evaluation used here against the oracle's whole-grid restriction."""
    nx, ny, nz = 8, 6, 6
    A = fine_stencil(nz, 1.0 / nz, LAM, MU)
    rng = np.random.default_rng(1)
    x, b = rng.standard_normal((2, 3, nz + 1, ny, nx))
    r = b - Level(nx, ny, nz, A).apply(x)
    r[:, [0, -1]] = 0
    whole = restrict(r)
    w, at = np.array([0.5, 1.0, 0.5]), np.arange(-2, 3)
    for K, J, I in ((1, 0, 0), (2, 2, 3), (1, 1, 2)):
        cut = lambda f: f[np.ix_(range(3), 2 * K + at, (2 * J + at) % ny, (2 * I + at) % nx)]  # noqa: E731
        p = cut(b) - Level(5, 5, 4, A[2 * K - 2:2 * K + 3]).apply(cut(x))
        v = np.einsum("cxyz,x,y,z->c", p[:, 1:4, 1:4, 1:4], w, w, w)
        assert np.allclose(v, whole[:, K, J, I], rtol=1e-12, atol=1e-9)


# coarse levels: 96 columns from three million values on (FP32: two nodes per
# thread, neighbours by lane), 20 columns (FP32: one node per thread), 64 columns
# (a row's pairs fill a run of lanes)
@pytest.mark.gpu
@pytest.mark.parametrize("n,coarse", [((192, 256, 192), 3), ((40, 24, 32), 4), ((128, 32, 32), 4)])
@pytest.mark.parametrize("precision", ["fp64", "fp32-ir"])
def test_coarse_level(n, coarse, precision):
    check(n, coarse, 1, precision)


# fine level, fused: planes per segment (FP64, FP32) and what is left for the last
@pytest.mark.gpu
@pytest.mark.parametrize("n,coarse", [
    ((96, 96, 96), 3),     # 3 with 2 left, 2 with 1 left
    ((128, 64, 96), 3),    # 2 with 1 left, 1
    ((192, 128, 64), 2),   # 4 with 3 left, 2 with 1 left
    ((72, 24, 16), 2),     # 1; tiles past the end of a row
    ((64, 8, 16), 4),      # 1; the tile's halo rows are its own
    ((6, 6, 4), 2),        # a single interior coarse plane
    ((768, 768, 64), 2)])  # 16 and 8, five rounds of resident workgroups
@pytest.mark.parametrize("precision", ["fp64", "fp32-ir"])
def test_fine_level(n, coarse, precision):
    check(n, coarse, 0, precision)
