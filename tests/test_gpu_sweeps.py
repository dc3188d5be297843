"""Single grids that the direction sweeps serve (more than 65536 nodes; smaller ones
step with tiles of both directions), ragged in both directions: every scheme against the
oracle, every tile shape, several steps in a call, stage-storing steps and the step
adjoint.  Bars as elsewhere: rhs 1e-12 of each component's maximum against the oracle,
one RK3 step 1e-11 of each component's increment; the rest bit for bit."""
import sys

import numpy as np
import pytest

from paper_1810_11103_amd import workloads as W
from test_gpu_parity import SCHEMES, STEPS_CASES, _dev, _host, make_case, normwise

pytestmark = pytest.mark.gpu
NX, NY = 301, 231


@pytest.fixture(scope="module")
def wiu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no ROCm device")
    from paper_1810_11103_amd import wenoiu
    assert wenoiu.tuning_applies(wenoiu.make_grid(NX, NY, (1, 1)), "5-2MP")
    return wenoiu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture
def shapes(wiu):
    """The selected tile shapes, put back afterwards."""
    saved = wiu.get_tuning(0), wiu.get_tuning(1)
    yield saved
    wiu.set_tuning(0, saved[0])
    wiu.set_tuning(1, saved[1])


@pytest.mark.parametrize("s", SCHEMES)
@pytest.mark.parametrize("kind", ["smooth", "riemann"])
def test_rhs_and_step_match_the_oracle(orc, wiu, s, kind):
    say("sweeps", s, kind)
    g, U = make_case(kind, NX, NY, seed=5)
    M = orc.metrics(s, g.x, g.y, g.bc, g.period)
    sol = wiu.Solver(g.x, g.y, s, g.bc, g.period)
    err = normwise(_host(sol.rhs(_dev(U))), orc.rhs(s, U, M, g.bc))
    assert np.all(err <= 1e-12), err
    dt = orc.cfl_dt(U, M, 0.5)
    Ud = _dev(U)
    sol.rk3_step_cfl(Ud, 0.5)
    assert float(sol.dt.item()) == pytest.approx(dt, rel=1e-13)
    err = normwise(_host(Ud) - U, orc.rk3_step(s, U, M, dt, g.bc) - U)
    assert np.all(err <= 1e-11), err
    assert sol.status() == 0


@pytest.mark.parametrize("s", SCHEMES)
def test_tile_shapes_give_identical_results(wiu, shapes, s):
    """Every pair of shapes: residual, and two steps, whose second and third stages take
    their line maxima from the eta tiles' lanes (2 to 16 lines per wave)."""
    say("sweeps: shapes", s)
    g, U = make_case("riemann", NX, NY, seed=4)
    sol = wiu.Solver(g.x, g.y, s, g.bc, g.period)
    Ud = _dev(U)
    ref = None
    for vx in range(wiu.tuning_variants(0)):
        for ve in range(wiu.tuning_variants(1)):
            wiu.set_tuning(0, vx)
            wiu.set_tuning(1, ve)
            r, V = sol.rhs(Ud), Ud.clone()
            sol.rk3_step(V, 2e-4)
            sol.rk3_step(V, 2e-4)
            ref = ref or (r, V)
            assert bool((r == ref[0]).all()) and bool((V == ref[1]).all()), (vx, ve)
    assert sol.status() == 0


def test_steps_cfl_across_tile_shapes(wiu, shapes):
    """The CFL maxima reduced in the eta tiles do not depend on their lane layout."""
    g, U = make_case("riemann", NX, NY, seed=9)
    sol = wiu.Solver(g.x, g.y, "5-2MP", g.bc, g.period)
    ref = None
    for ve in range(wiu.tuning_variants(1)):
        wiu.set_tuning(1, ve)
        Ud = _dev(U)
        out = sol.rk3_steps_cfl(Ud, 0.5, 3), Ud
        ref = ref or out
        assert bool((out[0] == ref[0]).all()) and bool((out[1] == ref[1]).all()), ve
    assert sol.status() == 0


@pytest.mark.parametrize("s,kind,sides,opts", STEPS_CASES)
def test_steps_cfl_equal_single_steps(wiu, s, kind, sides, opts):
    """Six steps go round the ring of four maxima sets more than once."""
    say("sweeps: steps_cfl", s, kind, sides, opts)
    g, U = make_case(kind, NX, NY, seed=8)
    sol = wiu.Solver(g.x, g.y, s, g.bc, g.period, params=wiu.make_params(**opts), sides=sides)
    Ua, Ub = _dev(U), _dev(U)
    dts = []
    for _ in range(6):
        sol.rk3_step_cfl(Ua, 0.5)
        dts.append(float(sol.dt.item()))
    assert _host(sol.rk3_steps_cfl(Ub, 0.5, 6)).tolist() == dts
    assert sol.status() == 0
    assert bool((Ua == Ub).all())


def test_steps_cfl_replayed_from_a_captured_graph(wiu):
    import torch
    say("sweeps: graph replays")
    g, U = make_case("riemann", NX, NY, seed=8)
    sol = wiu.Solver(g.x, g.y, "5-2MP", g.bc, g.period)
    U0 = _dev(U)
    K = 4
    Ue = U0.clone()
    dte = sol.rk3_steps_cfl(Ue, 0.5, K)
    Ug, dtg = U0.clone(), torch.empty(K, dtype=torch.float64, device="cuda")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sol.rk3_steps_cfl(Ug, 0.5, K, dtg)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sol.rk3_steps_cfl(Ug, 0.5, K, dtg)
    for r in range(3):
        Ug.copy_(U0)
        dtg.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Ug, Ue) and torch.equal(dtg, dte), r
        Uw = U0.clone()  # eager work between the replays
        sol.rk3_steps_cfl(Uw, 0.5, 2)
        torch.cuda.synchronize()
    assert sol.status() == 0


@pytest.mark.parametrize("s,kind,sides", [("5-2MP", "riemann", ("wall", "transmissive", "wall", "wall")),
                                          ("3-2MP", "smooth", None), ("7-4MP", "riemann", None)])
def test_steps_stages_equal_single_stage_steps(wiu, s, kind, sides):
    import torch
    say("sweeps: steps_stages", s, kind, sides)
    n = 5
    g, U = make_case(kind, NX, NY, seed=6)
    sol = wiu.Solver(g.x, g.y, s, g.bc, g.period, sides=sides)
    Ua, Ub = _dev(U), _dev(U)
    sol.cfl_dt(Ua, 0.4)
    Sa = torch.empty((n, 3) + U.shape, dtype=torch.float64, device="cuda")
    Sb = torch.empty_like(Sa)
    Ra, Rb = sol.step_record(n), sol.step_record(n)
    for k in range(n):
        Sa[k, 0].copy_(Ua)
        sol.rk3_step_stages(Ua, Sa[k, 1], Sa[k, 2], rec=Ra[k])
    sol.rk3_steps_stages(Ub, Sb, Rb)
    assert sol.status() == 0
    assert torch.equal(Ua, Ub) and torch.equal(Sa, Sb)
    ra, rb = (r.view(n, 3, -1)[:, :, :NX + NY] for r in (Ra, Rb))
    assert torch.equal(ra, rb)


@pytest.mark.parametrize("s", ["3-1MP", "5-2MP"])
def test_step_adjoint_with_recomputed_stages(orc, wiu, s):
    """From recomputed, stored and recorded stages alike, and against the oracle (bar
    1e-11 of each component's maximum, as on smaller grids)."""
    import torch
    say("sweeps: step adjoint", s)
    g, U = make_case("smooth", NX, NY, seed=7)
    sol = wiu.Solver(g.x, g.y, s, g.bc, g.period)
    Ud = _dev(U)
    M = orc.metrics(s, g.x, g.y, g.bc, g.period)
    dt = 0.5 * orc.cfl_dt(U, M, 0.5)
    Wt = np.random.default_rng(5).standard_normal(U.shape)
    sol.dt.fill_(dt)
    U1, U2, rec = torch.empty_like(Ud), torch.empty_like(Ud), sol.step_record()
    sol.rk3_step_stages(Ud.clone(), U1, U2, rec=rec)
    W_ = _dev(Wt)
    a = sol.rk3_step_vjp(Ud, W_)
    assert torch.equal(a, sol.rk3_step_vjp(Ud, W_, U1, U2))
    assert torch.equal(a, sol.rk3_step_vjp(Ud, W_, U1, U2, rec=rec))
    assert sol.status() == 0
    err = normwise(_host(a), orc.rk3_step_vjp(s, U, M, dt, Wt, g.bc))
    assert np.all(err <= 1e-11), err
