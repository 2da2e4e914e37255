"""A solution that a query or an adjoint on another stream still reads keeps its
memory until that stream has passed the call, although autograd lets go of the
solution at once: of the latest one when the next solve starts, of the others with
their graph."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2609_28458_amd import api, inputs  # noqa: E402
from paper_2609_28458_amd.autograd import SolveSpec, solve_ad  # noqa: E402


@pytest.mark.parametrize("explicit", [True, False], ids=["given", "current"])
@pytest.mark.parametrize("call", ["dense", "vjp"])
def test_memory_waits_for_the_other_stream(call, explicit):
    n, Q = 4096, 200
    w = inputs.orbits_forward(n=n, seed=91)
    spec = SolveSpec(w["rhs"], w["tableau"], 0.0, 20.0, 1e-8, 1e-10)
    y0 = torch.as_tensor(w["y0"], device="cuda").requires_grad_()
    th = torch.as_tensor(w["theta"], device="cuda")
    outs = solve_ad(spec, y0, th)
    sol = spec.last_solution
    tq = torch.as_tensor(np.random.default_rng(92).uniform(0.0, 20.0, (Q, n)), device="cuda")
    yb = torch.ones((1, 6, n), dtype=torch.float64, device="cuda")
    reps = 20 if call == "dense" else 30

    def queue(stream):
        if call == "dense":
            return [api.dense_eval(sol, tq, stream=stream) for _ in range(reps)]
        return [api.solve_vjp(sol, ybar_final=yb, stream=stream)[0] for _ in range(reps)]

    want = queue(None)[0]
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    if explicit:
        got = queue(side)
    else:
        with torch.cuda.stream(side):
            got = queue(None)
    end = torch.cuda.Event()
    end.record(side)
    place, size = sol.workspace.data_ptr(), sol.workspace.numel()
    del outs, sol
    spec.last_solution = None  # as the next solve does first
    # What a solve on this stream would be given next for a tape of this size.
    again = torch.empty(size, dtype=torch.uint8, device="cuda")
    assert not end.query(), "the other stream has to be still at work"
    assert again.data_ptr() != place
    again.fill_(255)
    torch.cuda.synchronize()
    for g in got:
        assert torch.equal(g, want)
