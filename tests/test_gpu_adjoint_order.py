"""An adjoint takes the library's own order only if the forward built it.  A
forward with a caller's order, on the static schedule or with a workspace too small
for the library's order leaves that place of the workspace as it was; an adjoint whose
arguments would call for the order then goes in index order, which any tape
serves, and its gradients are those of an index-order forward, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2609_28458_amd import api, inputs  # noqa: E402

N = 16_385  # one more than the least ensemble the library orders by itself


@pytest.mark.parametrize("left", [0xFF, 0x00], ids=["no index", "one index"])
@pytest.mark.parametrize("forward", ["caller", "static", "small workspace", "own"])
@pytest.mark.parametrize("k", [1, 8])
def test_adjoint_without_the_forwards_order(k, forward, left):
    w = {**inputs.orbits_uneven(N, seed=81), "t1": 2.0, "rtol": 1e-5, "atol": 1e-5}
    prob = api.make_problem(w["rhs"], w["tableau"], w["y0"], w["theta"], w["t0"], w["t1"],
                            w["rtol"], w["atol"])
    L = api.Launch(ckpt_every=k, ckpt_capacity=256 // k)
    yb = torch.as_tensor(np.random.default_rng(82).normal(size=(1, prob.d, N)), device="cuda")

    ref = api.Solution(prob, L)
    ref.set_order(np.arange(N))
    ref.run()
    want = api.solve_vjp(ref, ybar_final=yb)
    assert bool((ref.status == 0).all())

    sol = api.Solution(prob, L)
    sol.workspace.fill_(left)  # what the place of the order holds beforehand
    a, full = sol.args, sol.args.workspace_bytes
    if forward == "caller":
        sol.set_order(np.random.default_rng(83).permutation(N))
    elif forward == "static":
        a.schedule = api.SCHEDULE["static"]
    elif forward == "small workspace":
        a.workspace_bytes -= 8 * N + 256
    sol.run()
    a.schedule, a.workspace_bytes = api.SCHEDULE["queue"], full
    sol.set_order(None)
    for _ in range(2):  # the second one finds what the first one left
        got = api.solve_vjp(sol, ybar_final=yb)
        for g, r in zip(got, want):
            assert torch.equal(g, r)
        assert sol.replay_mismatches() == 0
