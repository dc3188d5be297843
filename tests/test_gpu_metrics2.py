"""2-D metrics at the edges of their kernel's tiles (32 x 16 nodes from the first
ghost node on, so 24 x 8 nodes fill one) for every reach of the central operators
(3 to 7 nodes) and both midpoint interpolations, on grids smaller than a stencil
too.  Bar: 1e-13 of each metric vector's magnitude, as for all metrics."""
import sys

import numpy as np
import pytest

from paper_1810_11103_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wiu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no ROCm device")
    from paper_1810_11103_amd import wenoiu
    return wenoiu


CASES = [("3-1MP", 24, 8, "periodic"), ("3-1MP", 2, 3, "bounded"), ("3-2MP", 23, 9, "bounded"),
         ("3-2MP", 25, 7, "periodic"), ("5-1MP", 56, 24, "bounded"), ("5-2MP", 57, 25, "bounded"),
         ("5-2MP", 55, 23, "periodic"), ("5-2MP", 1, 5, "periodic"), ("7-1MP", 24, 9, "bounded"),
         ("7-2MP", 89, 41, "periodic"), ("7-4MP", 2, 2, "bounded"), ("7-4MP", 71, 40, "bounded"),
         ("7-6MP", 5, 1, "periodic"), ("7-6MP", 74, 39, "bounded"), ("7-6MP", 121, 56, "periodic"),
         ("7-6MP", 31, 1, "strip")]


@pytest.mark.parametrize("s,nx,ny,kind", CASES)
def test_metrics_tile_edges(orc, wiu, s, nx, ny, kind):
    print("metrics2", s, nx, ny, kind, file=sys.stderr, flush=True)
    if kind == "periodic":
        g = W.periodic_grid(nx, ny, (0, 10, 0, 10), A=0.2, seed=4)
    elif kind == "bounded":
        g = W.bounded_grid(nx, ny, (0, 1, 0, 1), A=0.2, seed=5)
    else:
        g = W.strip_grid(nx)
    sol = wiu.Solver(g.x, g.y, s, g.bc, g.period)
    M = sol.planes().cpu().numpy()
    ref = orc.metrics(s, g.x, g.y, g.bc, g.period)
    for planes in [(0, 1), (2, 3), (4,), (5, 6), (7, 8)]:
        scale = max(np.abs(ref[p]).max() for p in planes)
        for p in planes:
            assert np.abs(M[p] - ref[p]).max() <= 1e-13 * scale, p
