"""One lane per trajectory under the queue schedule, for ensembles that go to groups
or tangent lanes by themselves: a grid too small for those keeps the single lanes (the
queue heads in the workspace show it), so their loop is run with every refill threshold,
with outputs, tapes, stops, invalid inputs and orders, and with dual numbers.
References, bit for bit: the static schedule and 16-lane groups, tangent lanes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import to_np  # noqa: E402
from paper_2609_28458_amd import api, inputs  # noqa: E402

N = 1500
GRIDS = (dict(grid=1, block=64), dict(grid=3, block=128), dict(grid=4))


def _prob(tab, outputs, stops=True, n=N):
    w = inputs.orbits_uneven(n, seed=121)
    y0, t1 = w["y0"].copy(), np.minimum(w["t1"], 6.0)
    rtol = np.broadcast_to(w["rtol"], (n,)).copy()
    if stops:
        y0[2, 5] = np.nan
        y0[0, n - 2] = np.inf
        t1[9] = 0.0         # an empty span
        t1[11] = -1.0       # bad input
        rtol[13] = 0.0      # bad input
    t_out = None
    if outputs == "shared":
        t_out = np.linspace(0.0, t1[t1 > 0.0].min(), 5)  # past the empty span: bad input
    elif outputs == "own":
        t_out = np.sort(np.random.default_rng(122).uniform(0.0, 1.0, (12, n)), axis=0)
        t_out[0] = 0.0
        t_out[-1, ::3] = 1.0                       # exactly at the end
        t_out = t_out * np.maximum(t1, 0.0)
    elif outputs == "outside":
        t_out = np.linspace(0.0, 6.0, 7)           # past some ends: bad input
    atol = np.broadcast_to(w["atol"], (n,)).copy()
    return api.make_problem(w["rhs"], tab, y0, w["theta"], 0.0, t1, rtol, atol, t_out)


def _run(prob, order=None, **launch):
    sol = api.Solution(prob, api.Launch(**launch))
    sol.workspace[:256] = 7
    if order is not None:
        sol.set_order(order, check=False)
    sol.run()
    torch.cuda.synchronize()
    return sol


def _heads(sol):
    h = sol.workspace[:32].view(torch.int64).cpu().numpy()
    return int(h[0]), int(h[3])


def _same(got, ref, rows=slice(None)):
    a, b = to_np(got), to_np(ref)
    for k in b:
        if k == "y_out" and got.launch.out_layout == "knd":
            a[k] = a[k].transpose(2, 0, 1)
        np.testing.assert_array_equal(a[k][..., rows], b[k][..., rows], err_msg=k)
    return b


@pytest.mark.parametrize("refill", [1, 8, 32, 64])
@pytest.mark.parametrize("outputs", ["none", "shared", "own", "outside"])
@pytest.mark.parametrize("tab", ["dopri5", "tsit5", "verner7"])
def test_queue_of_single_lanes(tab, outputs, refill):
    prob = _prob(tab, outputs)
    rng = np.random.default_rng(123)
    order = rng.permutation(N)
    for kw in (dict(), dict(max_steps=60)):
        ref = _run(prob, schedule="static", **kw)
        grp = _run(prob, wide=N, **kw)
        st = _same(grp, ref)["status"]
        assert {0, 3, 5} <= set(st.tolist()) if outputs != "outside" else np.any(st == 5)
        if kw:
            assert np.any(st == 1)
        for g in GRIDS:
            for extra in (dict(), dict(out_layout="knd")):
                sol = _run(prob, order=order, refill=refill, **g, **extra, **kw)
                lanes_head, groups_head = _heads(sol)
                assert lanes_head >= N and groups_head == 0
                _same(sol, ref)
    # an order with a repeated and a bad entry: one trajectory is left out
    bad = torch.as_tensor(order, device="cuda")
    left = int(bad[N // 2])
    bad[N // 2] = N + 7
    sol = _run(prob, order=bad, refill=refill, **GRIDS[1])
    assert int(sol.status[left]) == 6
    _same(sol, _run(prob, schedule="static"), rows=np.arange(N) != left)


@pytest.mark.parametrize("refill", [1, 8, 64])
@pytest.mark.parametrize("k", [1, 5])
@pytest.mark.parametrize("outputs", ["none", "own"])
@pytest.mark.parametrize("tab", ["dopri5", "verner7"])
def test_tape_of_single_lanes(tab, outputs, k, refill):
    """Tapes of two capacities (the smaller one overflows), and the gradients of both
    the solve's outputs and its final state."""
    prob = _prob(tab, outputs)
    full = int(_run(prob, schedule="static").n_accepted.max()) // k + 2
    yb = torch.as_tensor(np.random.default_rng(124).normal(size=(1, 6, N)), device="cuda")
    yo = (torch.as_tensor(np.random.default_rng(125).normal(size=(1, 6, prob.K, N)),
                          device="cuda") if prob.K else None)
    for cap in (full, full // 2):
        kw = dict(ckpt_every=k, ckpt_capacity=cap)
        ref = _run(prob, schedule="static", **kw)
        want = api.solve_vjp(ref, ybar_final=yb, ybar_out=yo)
        assert (4 in ref.status.tolist()) == (cap < full)
        for g in GRIDS:
            sol = _run(prob, refill=refill, **g, **kw)
            lanes_head, groups_head = _heads(sol)
            assert lanes_head >= N and groups_head == 0
            _same(sol, ref)
            got = api.solve_vjp(sol, ybar_final=yb, ybar_out=yo, grid=3)
            for a, b in zip(got, want):
                np.testing.assert_array_equal(a.cpu().numpy(), b.cpu().numpy())
            assert sol.replay_mismatches() == 0


@pytest.mark.parametrize("refill", [1, 32, 64])
@pytest.mark.parametrize("tab,outputs", [("dopri5", "own"), ("tsit5", "shared"), ("dopri5", "none"),
                                         ("verner7", "none")])
def test_dual_numbers_in_one_lane(tab, outputs, refill):
    """Four columns, two launches: on this grid a lane each, with stops and invalid
    trajectories; tangent lanes are the reference."""
    prob = _prob(tab, outputs)
    cols = [6, 0, 7, 2]
    order = np.random.default_rng(126).permutation(N)
    for kw in (dict(), dict(max_steps=60)):
        ref, R, RO = api.solve_sens(prob, cols, api.Launch(**kw))
        for g in GRIDS:
            sol, S, SO = api.solve_sens(prob, cols, api.Launch(refill=refill, **g, **kw),
                                        order=order)
            torch.cuda.synchronize()
            assert N <= _heads(sol)[0] < 2 * N  # on tangent lanes two groups an orbit
            st = _same(sol, ref)["status"]
            assert (1 in st) == bool(kw) and {3, 5} <= set(st.tolist())
            np.testing.assert_array_equal(S.cpu().numpy(), R.cpu().numpy())
            if SO is not None:
                np.testing.assert_array_equal(SO.cpu().numpy(), RO.cpu().numpy())


@pytest.mark.parametrize("n,K", [(3, 8), (5, 9), (65, 8), (131, 0)])
@pytest.mark.parametrize("tab", ["dopri5", "verner7"])
def test_groups_from_their_queue(tab, n, K):
    """Every trajectory on groups of a grid that holds four of them, with outputs in
    the loop and deferred."""
    w = inputs.quintessence(n, seed=127)
    t_out = np.linspace(w["t0"], w["t1"], K) if K else None
    prob = api.make_problem(w["rhs"], tab, w["y0"], w["theta"], w["t0"], w["t1"], w["rtol"],
                            w["atol"], t_out)
    sol = _run(prob, grid=1, block=64, wide=n)
    assert n <= 4 or _heads(sol)[1] >= n
    _same(sol, _run(prob, schedule="static"))
    _same(_run(prob), _run(prob, schedule="static"))


@pytest.mark.parametrize("n,M", [(5, 1), (33, 3), (65, 4)])
def test_tangent_lanes_from_their_queue(n, M):
    """Systems whose tangents do not fit one lane take tangent lanes on any grid."""
    w = inputs.spin_precession(n, seed=128)
    prob = api.make_problem(w["rhs"], "dopri5", w["y0"], w["theta"], 12.0 ** -0.5, w["t1"], 1e-6,
                            1e-8, np.array([11.0 ** -0.5]))
    cols = [9, 10, 0, 11][:M]
    a, Sa, Oa = api.solve_sens(prob, cols, api.Launch())
    b, Sb, Ob = api.solve_sens(prob, cols, api.Launch(grid=1, block=64))
    torch.cuda.synchronize()
    _same(b, a)
    assert torch.equal(Sa, Sb) and torch.equal(Oa, Ob)
