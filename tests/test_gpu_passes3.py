"""3-D passes on both sides of the grid size from which the zeta and eta passes run
one after the other instead of side by side (2^21 nodes), with tiles of 30 items where
a line has as many segments of them as of 32, else of 32: a grid that repeats a
smaller one ten times along k has the smaller one's residual in every period, and a
step's increments.  Bar 1e-11 of each component's maximum: the repeated coordinates
carry 2^-53 of ten periods, 1.4e-14 of a cell's size, and the residual is a difference
of fluxes up to a hundred times itself."""
import sys

import numpy as np
import pytest

from paper_1810_11103_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s,n,kw", [("5-2MP", (130, 126, 13), {}), ("3-1MP", (64, 257, 13), {}),
                                    ("5-2MP", (128, 140, 13), {}), ("5-1MP", (66, 262, 13), {}),
                                    ("7-2MP", (128, 128, 13), {"vars": "primitive"})])
def test_repeated_grid(s, n, kw):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no ROCm device")
    from paper_1810_11103_amd import wenoiu
    print("passes3", s, n, kw, file=sys.stderr, flush=True)
    g = W.periodic_grid3(*n, box=(0.0, 2.0, 0.0, 2.0, 0.0, 1.0), A=0.1, seed=2)
    U = W.smooth_state3(g, seed=3)
    rep = lambda a: np.concatenate([a] * 10, axis=-3)
    z = np.concatenate([g.z + q * g.period[2] for q in range(10)])
    out = []
    for x, y, z_, period, U_ in [(g.x, g.y, g.z, g.period, U),
                                 (rep(g.x), rep(g.y), z, g.period[:2] + (10 * g.period[2],), rep(U))]:
        sol = wenoiu.Solver3(x, y, z_, s, g.bc, period, params=wenoiu.make_params(**kw))
        Ud = torch.as_tensor(np.ascontiguousarray(U_), dtype=torch.float64).cuda()
        r = sol.rhs(Ud)
        U1 = Ud.clone()
        sol.rk3_step_cfl(U1, 0.5)
        out.append((r, U1 - Ud))
    small = out[0][0].numel() // 5
    assert small < 2 ** 21 <= 10 * small
    for a, b in zip(*out):
        for c in range(5):
            scale = float(a[c].abs().max())
            for q in range(10):
                d = float((b[c, q * n[2]:(q + 1) * n[2]] - a[c]).abs().max())
                assert d <= 1e-11 * scale, (c, q, d / scale)
