"""The equations do not change when density, momentum and energy are multiplied by one
number: the residual is multiplied by it too and its adjoint stays.  With a power of
two that holds bit for bit as long as nothing over- or underflows, so it shows the range
of states that the weights take.  The largest numbers formed are their sums: 2^2, 2^4 and
2^6 times the fourth (r = 2), eighth (r = 3) and twelfth (r = 4) powers of second
differences of up to 2^2.5 times the number (a little more in 3-D), to stay below
2^1024.  The smallest are the indicators, above 2^-39 times its square here, to which
the epsilon of 2^-133 adds nothing down to 2^-20."""
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


def rough(shape, seed=1):
    rng = np.random.default_rng(seed)
    D = len(shape)
    U = np.empty((D + 2,) + shape)
    U[0] = 1 + 0.4 * rng.random(shape)
    U[1:-1] = 0.5 * rng.standard_normal((D,) + shape)
    U[-1] = 2.5 + rng.random(shape) + 0.5 * (U[1:-1] ** 2).sum(0) / U[0]
    return U


@pytest.mark.parametrize("s,k", [("3-1MP", 252), ("5-2MP", 125), ("7-4MP", 81)])
@pytest.mark.parametrize("nx,ny", [(40, 36), (300, 230)])  # stage tiles, sweeps
@pytest.mark.parametrize("kw", [{}, {"ppm": 0}, {"weights": "z"}])
def test_scaled_state(wiu, s, k, nx, ny, kw):
    import torch
    print("range", s, nx, ny, kw, file=sys.stderr, flush=True)
    if "weights" in kw:  # products of the indicators themselves, not of their squares
        k = {2: 253, 3: 168, 4: 124}[(int(s[0]) + 1) // 2]
    g = W.periodic_grid(nx, ny, (0, 10, 0, 10), A=0.2, seed=3)
    U = torch.as_tensor(rough((36, 40))).cuda()
    U = U.repeat(1, -(-ny // 36), -(-nx // 40))[:, :ny, :nx].contiguous()
    sol = wiu.Solver(g.x, g.y, s, g.bc, g.period, params=wiu.make_params(**kw))
    r = sol.rhs(U)
    for q in (-20, k):
        assert bool((sol.rhs(U * 2.0 ** q) == r * 2.0 ** q).all()), q
    if s[0] != "7" and "weights" not in kw:
        G = torch.as_tensor(np.random.default_rng(2).standard_normal(U.shape)).cuda()
        v = sol.rhs_vjp(U, G)
        assert bool((sol.rhs_vjp(U * 2.0 ** k, G) == v).all())


@pytest.mark.parametrize("s,k", [("3-1MP", 252), ("5-2MP", 124), ("7-4MP", 80)])
def test_scaled_state_3d(wiu, s, k):
    import torch
    print("range 3-D", s, file=sys.stderr, flush=True)
    g = W.periodic_grid3(20, 18, 16, box=(0.0, 2.0, 0.0, 1.0, 0.0, 3.0), A=0.2, seed=4)
    U = torch.as_tensor(rough((16, 18, 20))).cuda()
    sol = wiu.Solver3(g.x, g.y, g.z, s, g.bc, g.period)
    r = sol.rhs(U)
    for q in (-20, k):
        assert bool((sol.rhs(U * 2.0 ** q) == r * 2.0 ** q).all()), q
