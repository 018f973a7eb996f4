"""GPU: what qs_setup costs for a hierarchy of three levels, whose two coarsest
are prepared as one map."""
import time

import pytest

torch = pytest.importorskip("torch")

from workloads import lame

pytestmark = pytest.mark.gpu
LAM, MU = lame()


def setup_seconds(n, coarse, precision):
    from paper_1904_03808_amd.qsmg import MGSolver
    best = 1e9
    for _ in range(10):
        torch.cuda.synchronize()
        t = time.perf_counter()
        g = MGSolver(n, n, n, 1.0 / n, LAM, MU, min_coarse_nz=coarse, precision=precision)
        torch.cuda.synchronize()
        best = min(best, time.perf_counter() - t)
        g.close()
    return best


@pytest.mark.parametrize("precision", ["fp64", "fp32-ir"])
def test_map_is_cheap_to_prepare(precision):
    """16^3 down to 4^3 against 8^3 down to 4^3, which has the same coarsest inverse
    and no map: a setup is a few dozen uploads and launches either way, so three
    times the time bounds it (one cycle per unknown of the map, 84 of them, is ten)."""
    setup_seconds(8, 4, precision)
    assert setup_seconds(16, 4, precision) <= 3 * setup_seconds(8, 4, precision)
