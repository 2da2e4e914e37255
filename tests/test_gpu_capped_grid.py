"""A caller's grid holds what it did with one lane per trajectory: groups and
tangent lanes are chosen by themselves only where that grid holds them, and a grid
without a block counts workgroups of four wavefronts.  Which way a solve went shows in
the queue heads of its workspace: the single lanes' (word 0) and the groups' (word 3), or
neither where every trajectory has its own place."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import to_np  # noqa: E402
from paper_2609_28458_amd import api, inputs  # noqa: E402

N = 4096
UNTOUCHED = 0x0707070707070707


def _prob(n=N, tab="dopri5", t1=4.0):
    w = inputs.orbits_forward(n, seed=101)
    return api.make_problem(w["rhs"], tab, w["y0"], w["theta"], 0.0, t1, 1e-7, 1e-9)


def _heads(sol):
    torch.cuda.synchronize()
    h = sol.workspace[:32].view(torch.int64).cpu().numpy()
    return int(h[0]), int(h[3])


def _run(prob, **launch):
    sol = api.Solution(prob, api.Launch(**launch))
    sol.workspace[:256] = 7
    return sol.run()


@pytest.mark.parametrize("launch,groups", [
    (dict(block=256, grid=16), False), (dict(grid=16), False), (dict(block=64, grid=64), False),
    (dict(grid=255), False), (dict(grid=256), True), (dict(block=64, grid=1024), True),
    (dict(block=64), True), (dict(), True)])
def test_groups_only_where_the_grid_holds_them(launch, groups):
    prob = _prob()
    sol = _run(prob, **launch)
    lanes_head, groups_head = _heads(sol)
    if groups:
        assert lanes_head == groups_head == UNTOUCHED
    else:
        assert lanes_head >= N and groups_head == 0
    a, b = to_np(sol), to_np(api.solve(prob, api.Launch(schedule="static")))
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)


@pytest.mark.parametrize("launch,head", [(dict(grid=16), False), (dict(grid=256), True),
                                         (dict(), True)])
def test_head_of_the_own_order_on_a_grid(launch, head):
    n = 17_000
    sol = _run(_prob(n, t1=1.0), ckpt_every=1, ckpt_capacity=256, **launch)
    lanes_head, groups_head = _heads(sol)
    assert lanes_head >= n and (groups_head >= 512 if head else groups_head == 0)


# Four columns: eight tangent lanes an orbit against two launches of one lane;
# nine: twelve against five.
@pytest.mark.parametrize("M,launch,tangent_lanes", [
    (4, dict(grid=16), False), (4, dict(block=256, grid=16), False), (9, dict(grid=16), True),
    (4, dict(), True)])
def test_tangent_lanes_only_where_the_grid_holds_them(M, launch, tangent_lanes):
    prob = _prob(tab="tsit5")
    cols = list(range(M))
    sol, S, _ = api.solve_sens(prob, cols, api.Launch(**launch))
    lanes_head, _ = _heads(sol)
    chunks = (M + 2) // 3
    if launch:
        assert (lanes_head >= chunks * N) == tangent_lanes
    ref, R, _ = api.solve_sens(prob, cols, api.Launch())
    torch.cuda.synchronize()
    assert torch.equal(S, R) and torch.equal(sol.y_final, ref.y_final)


def _ms(fn):
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    fn()
    times = []
    for _ in range(7):
        ev[0].record()
        fn()
        ev[1].record()
        torch.cuda.synchronize()
        times.append(ev[0].elapsed_time(ev[1]))
    return min(times)


@pytest.mark.parametrize("call", ["solve", "sens", "vjp"])
def test_grid_without_a_block_holds_four_wavefronts_each(call):
    prob = _prob(t1=20.0, tab="tsit5")
    if call == "solve":
        def run(**kw):
            sol = api.Solution(prob, api.Launch(grid=16, **kw))
            return sol.run
    elif call == "sens":
        def run(**kw):
            return lambda: api.solve_sens(prob, [6, 7], api.Launch(grid=16, **kw))
    else:
        sol = api.solve(prob, api.Launch(ckpt_every=1, ckpt_capacity=2000))
        yb = torch.ones((1, 6, N), dtype=torch.float64, device="cuda")

        def run(**kw):
            return lambda: api.solve_vjp(sol, ybar_final=yb, grid=16, **kw)
    # The same launch, named and not: four rounds of a quarter of the lanes take
    # 1.8 to 3 times as long.
    assert _ms(run()) < 1.3 * _ms(run(block=256))
