"""Which tile shape a sweep is launched with: the names of the kernels that ran."""
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


def kernels(f):
    import torch
    from torch.profiler import ProfilerActivity, profile
    f()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as p:
        f()
        torch.cuda.synchronize()
    return [e.name for e in p.events() if "wiu::" in e.name]


def problem(wiu, nx, ny, s="5-2MP"):
    import torch
    print("tuning", s, nx, ny, file=sys.stderr, flush=True)
    g = W.periodic_grid(nx, ny, (0, 10, 0, 10), A=0.1, seed=3)
    U = torch.as_tensor(np.ascontiguousarray(W.random_smooth_state(g, seed=5))).cuda()
    return wiu.Solver(g.x, g.y, s, g.bc, g.period), U


def xi_tiles(wiu, sol, U):
    names = kernels(lambda: sol.rhs(U))
    return [n.split("<")[1].split(">")[0].replace(" ", "").split(",")[2:4] for n in names if "sweep_kernel<" in n and
            n.split("<")[1].replace(" ", "").split(",")[1] == "0"]


def test_a_selection_that_is_put_back_is_the_first(wiu):
    """Saving the selection, changing it and putting it back leaves the choice by the
    grid as it was: 64 x 2 on 300 columns, 128 x 1 on 2048."""
    a, b = problem(wiu, 300, 400), problem(wiu, 2048, 40)
    first = xi_tiles(wiu, *a), xi_tiles(wiu, *b)
    assert first == ([["64", "2"]], [["128", "1"]])
    saved = wiu.get_tuning(0)
    try:
        wiu.set_tuning(0, 1)
        assert xi_tiles(wiu, *a) == [["256", "1"]]
        wiu.set_tuning(0, 2)
        assert xi_tiles(wiu, *b) == [["64", "2"]]
    finally:
        wiu.set_tuning(0, saved)
    assert (xi_tiles(wiu, *a), xi_tiles(wiu, *b)) == first


def test_tuning_a_grid_of_stage_tiles_changes_nothing(wiu, tmp_path):
    from paper_1810_11103_amd import autotune
    cache = tmp_path / "tuning.json"
    before = wiu.get_tuning(0), wiu.get_tuning(1)
    sol, U = problem(wiu, 200, 180)
    assert not wiu.tuning_applies(sol.grid, "5-2MP")
    assert not any("sweep_kernel" in n for n in kernels(lambda: sol.rhs(U)))
    try:
        res = autotune.tune_single(sol, U, cache=str(cache))
        assert tuple(res["variant"]) == before == (wiu.get_tuning(0), wiu.get_tuning(1))
        assert res["ms"] > 0.0 and not cache.exists()
        sol, U = problem(wiu, 300, 230)
        assert wiu.tuning_applies(sol.grid, "5-2MP")
        res = autotune.tune_single(sol, U, cache=str(cache))
        assert tuple(res["variant"]) == (wiu.get_tuning(0), wiu.get_tuning(1))
        assert len(res["all_ms"]) == wiu.tuning_variants(0) * wiu.tuning_variants(1) and cache.exists()
    finally:
        wiu.set_tuning(0, before[0])
        wiu.set_tuning(1, before[1])


@pytest.mark.parametrize("s", ["3-1MP", "3-2MP", "5-1MP", "5-2MP", "7-1MP", "7-2MP", "7-4MP", "7-6MP"])
def test_shape_of_a_batch_counts_the_lanes_that_run(wiu, s):
    """The rule for a batch knows how many tiles either shape gives (128 lanes each)."""
    blocks = []
    for nx, ny in [(40, 31), (125, 24), (121, 17), (59, 30), (57, 9), (1, 5)]:
        g = W.periodic_grid(nx, ny, (0, 10, 0, 10), A=0.1, seed=3)
        blocks.append((g.x, g.y, g.bc, g.period))
    for some in (blocks, blocks[1:2], blocks[2:3], blocks[4:5], blocks[5:]):
        n = {v: wiu.BatchedPlan(some, s, xi_variant=v).info()[1] for v in (0, 2)}
        plan = wiu.BatchedPlan(some, s)
        assert plan.variant[0] == (2 if n[2] <= n[0] else 0), n
        assert plan.info()[1] == min(n.values())
