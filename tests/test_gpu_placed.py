"""Launches that hold every trajectory on a group take the positions of the
order by place: ensembles at the ends of wavefronts (4 groups), with an order
that reverses the trajectories and leaves one out, a grid too small to hold them
all, and the output counts up to which outputs are evaluated in the loop.  One lane
per trajectory (the static schedule) is the reference, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import to_np  # noqa: E402
from paper_2609_28458_amd import api, inputs  # noqa: E402


def _run(prob, order=None, **launch):
    sol = api.Solution(prob, api.Launch(**launch))
    sol.workspace.fill_(7)  # nothing is read that the solve did not write
    if order is not None:
        sol.set_order(order, check=False)
    sol.run()
    torch.cuda.synchronize()
    assert sol.replay_mismatches() == 0
    return to_np(sol)


@pytest.mark.parametrize("n,K", [(1, 0), (3, 8), (4, 9), (5, 1), (16, 8), (17, 9), (511, 8)])
@pytest.mark.parametrize("tableau", ["dopri5", "tsit5", "verner7"])
def test_groups_by_place(tableau, n, K):
    w = inputs.quintessence(n, seed=61)
    t_out = np.linspace(w["t0"], w["t1"], K) if K else None
    prob = api.make_problem(w["rhs"], tableau, w["y0"], w["theta"], w["t0"], w["t1"], w["rtol"],
                            w["atol"], t_out)
    ref = _run(prob, schedule="static")
    assert np.all(ref["status"] == 0)
    order = torch.arange(n - 1, -1, -1, dtype=torch.int64, device="cuda")
    for got in (_run(prob), _run(prob, order=order), _run(prob, grid=1, block=64)):
        for k in ref:
            np.testing.assert_array_equal(got[k], ref[k], err_msg=k)
    if n > 1:
        order[n // 2] = -1  # leaves trajectory n - 1 - n // 2 out
        got, out = _run(prob, order=order), n - 1 - n // 2
        ran = np.arange(n) != out
        assert got["status"][out] == 6  # not run
        np.testing.assert_array_equal(got["y_final"][:, ran], ref["y_final"][:, ran])
        np.testing.assert_array_equal(got["n_accepted"][ran], ref["n_accepted"][ran])


@pytest.mark.parametrize("n,cols", [(1, 1), (31, 2), (33, 3), (65, 4)])
def test_tangent_lanes_by_place(n, cols):
    """Groups of 2 and 4 lanes: all at once against a grid of one workgroup,
    which takes them from the queue."""
    w = inputs.streams(n, seed=62)
    prob = api.make_problem(w["rhs"], w["tableau"], w["y0"], w["theta"], w["t0"], w["t1"],
                            w["rtol"], w["atol"])
    cols = [6, 7, 0, 3][:cols]
    a, Sa, _ = api.solve_sens(prob, cols, api.Launch())
    b, Sb, _ = api.solve_sens(prob, cols, api.Launch(grid=1, block=64))
    torch.cuda.synchronize()
    na, nb = to_np(a), to_np(b)
    for k in na:
        np.testing.assert_array_equal(na[k], nb[k], err_msg=k)
    assert torch.equal(Sa, Sb)
    assert a.replay_mismatches() == 0
