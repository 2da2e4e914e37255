"""What the library chooses by itself changes no bit: small ensembles on
16-lane groups and workgroups of one wavefront against one lane per trajectory
(the static schedule), and the library's own longest-first order of precessing
binaries against index order."""
import ctypes as C

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import to_np  # noqa: E402
from paper_2609_28458_amd import api, inputs  # noqa: E402


def _prob(w, n):
    th = w["theta"] if np.ndim(w["theta"]) == 1 else w["theta"][:, :n]
    return api.make_problem(w["rhs"], w["tableau"], w["y0"][:, :n], th, w["t0"], w["t1"],
                            w["rtol"], w["atol"], w["t_out"])


def _same(a, b):
    torch.cuda.synchronize()
    a, b = to_np(a), to_np(b)
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
    return a


# around the last size on groups (512 and 4,096 on 256 CUs) and the last one in
# workgroups of one wavefront (24,576)
@pytest.mark.parametrize("n", [1, 511, 512, 513, 4095, 4096, 4097, 24576, 24577])
@pytest.mark.parametrize("rhs", ["loghalo", "quint", "spinprec"])
def test_automatic_launch_equals_one_lane_each(rhs, n):
    api.lib()
    if rhs == "loghalo":
        w = inputs.orbits_forward(n, seed=51)
        w.update(t1=4.0, t_out=np.array([0.0, 1.3, 1.31, 4.0]), rtol=1e-6)
    elif rhs == "quint":
        w = inputs.quintessence(n, seed=51)
    else:
        w = inputs.spin_precession(n, seed=51)
        w.update(t0=14.0 ** -0.5, t_out=np.array([13.0 ** -0.5, 0.3]))
    g = _same(api.solve(_prob(w, n)), api.solve(_prob(w, n), api.Launch(schedule="static")))
    assert np.all(g["status"] == 0)


def test_own_order_of_binaries_changes_nothing():
    """More binaries than the launch holds (65,536 lanes at one wavefront per
    SIMD): the library's order, a workspace too small for it, and one lane each
    in index order give the same bits."""
    n = 66_001
    w = inputs.spin_precession(n, seed=52)
    w.update(t0=12.0 ** -0.5, t_out=None)
    prob = _prob(w, n)
    own = api.Solution(prob, api.Launch())
    assert own.args.workspace_bytes > 256 + 20 * n
    own.run()
    small = api.Solution(prob, api.Launch())
    small.args.workspace_bytes = 256
    small.run()
    _same(own, small)
    g = _same(own, api.solve(prob, api.Launch(schedule="static")))
    assert np.all(g["status"] == 0)
    # a sensitivity solve takes four lanes per binary, so it refills sooner
    m = 22_000
    p2 = _prob(w, m)
    a, Sa, _ = api.solve_sens(p2, [9, 10, 11])
    b, Sb, _ = api.solve_sens(p2, [9, 10, 11], order=np.arange(m)[::-1].copy())
    _same(a, b)
    assert torch.equal(Sa, Sb)


def test_order_of_binaries_follows_the_faster_spin():
    n = 5000
    w = inputs.spin_precession(n, seed=53)
    w["t_out"] = None
    w["theta"][0, :100] = 1.0 / w["theta"][0, :100]  # q > 1: the first spin is the faster
    sol = api.Solution(_prob(w, n), api.Launch())
    order = sol.queue_order().cpu().numpy()
    assert np.array_equal(np.sort(order), np.arange(n))
    q = w["theta"][0]
    key = np.log(4.0 + 3.0 * np.maximum(q, 1.0 / q))[order]
    width = (key.max() - key.min()) / 65534
    assert np.all(np.diff(key) <= width * (1 + 1e-9) + 1e-12)
    # without theta the span stands in, as for the other systems
    a = sol.args
    a.theta = None
    ws = torch.empty(api.gs_queue_order_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    assert api.lib().gs_queue_order(C.byref(a), None, out.data_ptr(), ws.data_ptr(),
                                    ws.numel()) == 0
    assert np.array_equal(np.sort(out.cpu().numpy()), np.arange(n))


@pytest.mark.parametrize("k", [1, 8])
@pytest.mark.parametrize("rhs", ["loghalo", "spinprec"])
def test_own_order_of_a_tape_changes_no_gradient(rhs, k):
    """With a tape of 256 steps or more the library orders 16,384 orbits or
    binaries by itself, forward and adjoint (orbits with the longest on
    groups): bitwise the gradients of index order, given or for want of room
    in the workspace."""
    n = 16_384
    if rhs == "loghalo":
        w = {**inputs.orbits_uneven(n, seed=54), "t1": 3.0, "rtol": 1e-6, "atol": 1e-6}
    else:
        w = {**inputs.spin_precession(n, seed=54), "t0": 11.0 ** -0.5, "t_out": None}
    prob = _prob(w, n)
    L = api.Launch(ckpt_every=k, ckpt_capacity=256 // k)
    yb = torch.as_tensor(np.random.default_rng(55).normal(size=(1, prob.d, n)), device="cuda")
    grads = []
    for how in ("own", "small workspace", "index order"):
        sol = api.Solution(prob, L)
        if how == "small workspace":
            sol.args.workspace_bytes -= 8 * n + 256  # cuts into the order's room at its end
        elif how == "index order":
            sol.set_order(np.arange(n))
        sol.run()
        grads.append(api.solve_vjp(sol, ybar_final=yb))
        assert bool((sol.status == 0).all())
        assert sol.replay_mismatches() == 0
    for other in grads[1:]:
        for a, b in zip(grads[0], other):
            assert torch.equal(a, b)


def test_differentiable_solve_frees_its_tape_with_its_outputs():
    """Nothing keeps a solution (and its tape) alive once the caller's tensors
    are gone, without the cycle collector; the next call starts by letting go
    of the latest one."""
    import gc
    import weakref

    from paper_2609_28458_amd.autograd import SolveSpec, solve_ad

    w = inputs.orbits_forward(n=64, seed=56)
    y0 = torch.as_tensor(w["y0"], device="cuda").requires_grad_()
    th = torch.as_tensor(w["theta"], device="cuda").requires_grad_()
    spec = SolveSpec(w["rhs"], w["tableau"], 0.0, 2.0, 1e-6, 1e-8, np.array([1.0, 2.0]))
    gc.disable()
    try:
        y_out, y_final, _ = solve_ad(spec, y0, th)
        first = weakref.ref(spec.last_solution)
        assert torch.equal(first().y_final, y_final) and not first().y_final.requires_grad
        (y_out.square().sum() + y_final.sum()).backward()
        spec.last_solution = None
        assert first() is not None  # the graph holds it
        del y_out, y_final
        assert first() is None
    finally:
        gc.enable()
