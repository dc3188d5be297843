"""Weights without the mapping (ppm = 0), whose kernels are compiled by themselves:
stage tiles, sweeps, batched sweeps and 3-D passes of every order against the oracle,
and the options' kernels, where the mapping is a test at run time.  Bars as elsewhere:
rhs 1e-12 of each component's maximum, one RK3 step 1e-11 of each component's
increment, a batched step 1e-11 likewise."""
import sys

import numpy as np
import pytest

from paper_1810_11103_amd import workloads as W
from test_gpu_3d import normwise
from test_gpu_parity import _dev, _host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def wiu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no ROCm device")
    from paper_1810_11103_amd import wenoiu
    return wenoiu


def say(*a):
    print("unmapped", *a, file=sys.stderr, flush=True)


@pytest.mark.parametrize("s", ["3-1MP", "3-2MP", "5-1MP", "5-2MP", "7-2MP", "7-4MP"])
@pytest.mark.parametrize("nx,ny,kw", [(61, 43, {}), (301, 231, {}), (61, 43, {"vars": "primitive"}),
                                      (301, 231, {"vars": "primitive"})])
def test_rhs_and_step(orc, wiu, s, nx, ny, kw):
    say(s, nx, ny, kw)
    g = W.periodic_grid(nx, ny, (0, 10, 0, 10), A=0.2, seed=3)
    U = W.random_smooth_state(g, seed=5)
    M = orc.metrics(s, g.x, g.y, g.bc, g.period)
    sol = wiu.Solver(g.x, g.y, s, g.bc, g.period, params=wiu.make_params(ppm=0, **kw))
    ref = orc.rhs(s, U, M, g.bc, ppm=0, **kw)
    # the mapping shows: its residual is another one
    assert np.all(normwise(orc.rhs(s, U, M, g.bc, **kw), ref) > 1e-9)
    err = normwise(_host(sol.rhs(_dev(U))), ref)
    assert np.all(err <= 1e-12), err
    dt = orc.cfl_dt(U, M, 0.5)
    Ud = _dev(U)
    sol.rk3_step(Ud, dt)
    err = normwise(_host(Ud) - U, orc.rk3_step(s, U, M, dt, g.bc, ppm=0, **kw) - U)
    assert np.all(err <= 1e-11), err
    assert sol.status() == 0


@pytest.mark.parametrize("s,kw", [("3-2MP", {}), ("5-2MP", {}), ("7-1MP", {}), ("5-1MP", {"vars": "conservative"})])
def test_batched_step(orc, wiu, s, kw):
    import torch
    say("batched", s, kw)
    blocks = W.batched_blocks(nblocks=4, seed=7, nmin=16, nmax=90)
    plan = wiu.BatchedPlan([(g.x, g.y, g.bc, g.period) for g, _ in blocks], s, params=wiu.make_params(ppm=0, **kw))
    for b, (_, U) in enumerate(blocks):
        plan.state(b).copy_(torch.as_tensor(U))
    plan.cfl_dt(0.4)
    dts = plan.get_dt()
    plan.step(graph=False)
    assert plan.status() == 0
    for b, (g, U) in enumerate(blocks):
        M = orc.metrics(s, g.x, g.y, g.bc, g.period)
        ref = orc.rk3_step(s, U, M, dts[b], g.bc, ppm=0, **kw) - U
        err = normwise(plan.state(b).cpu().numpy() - U, ref)
        assert np.all(err <= 1e-11), (b, err)
    plan.close()


@pytest.mark.parametrize("s,kw", [("3-1MP", {}), ("5-2MP", {}), ("7-2MP", {}), ("5-1MP", {"vars": "primitive"})])
def test_three_dimensions(orc, wiu, s, kw):
    say("3-D", s, kw)
    g = W.periodic_grid3(40, 36, 30, box=(0.0, 1.0, 0.0, 0.9, 0.0, 0.75), A=0.3, seed=3)
    U = W.smooth_state3(g, seed=3)
    M = orc.metrics3(s, g.x, g.y, g.z, g.bc, g.period)
    sol = wiu.Solver3(g.x, g.y, g.z, s, g.bc, g.period, params=wiu.make_params(ppm=0, **kw))
    ref = orc.rhs3(s, U, M, g.bc, ppm=0, **kw)
    assert np.all(normwise(orc.rhs3(s, U, M, g.bc, **kw), ref) > 1e-9)
    err = normwise(_host(sol.rhs(_dev(U))), ref)
    assert np.all(err <= 1e-12), err
    dt = orc.cfl_dt3(U, M, 0.5)
    Ud = _dev(U)
    sol.rk3_step(Ud, dt)
    err = normwise(_host(Ud) - U, orc.rk3_step3(s, U, M, dt, g.bc, ppm=0, **kw) - U)
    assert np.all(err <= 1e-11), err
    assert sol.status() == 0
